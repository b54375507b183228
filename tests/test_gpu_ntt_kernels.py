"""Every kernel of the transform multiply that bigint_mul and bigint_mullo can
pick, by name: each row says which transform its batch has to take
(bigint_mul_transform), at the largest operands that fit it, at unequal and odd
ones and just above the next smaller transform.  Through the C entries, with a
workspace only where the quarters take one; operands and results at odd limb
addresses, with guard limbs around the result.  Every product against the
MFMA-split multiply, the first four (all ones, zeros, long runs) against the
oracle; integers throughout, so the bytes are equal."""
import ctypes

import numpy as np
import pytest

from gpu_util import host, oracle_map, rand_limbs

pytestmark = pytest.mark.gpu

# points, way, na, nb, batch
FULL = [
    (2048, "side", 1024, 1024, 100), (2048, "side", 1061, 986, 100), (2048, "side", 1280, 767, 150),
    (3072, "serial", 1536, 1536, 2000), (3072, "serial", 1920, 1151, 3000),
    (3072, "side", 1536, 1536, 64), (3072, "side", 1573, 1498, 64), (3072, "side", 1250, 1201, 200),
    (4096, "side", 2048, 2048, 64), (4096, "side", 2560, 1535, 64), (4096, "side", 1537, 1536, 150),
    (5120, "serial", 2560, 2560, 1000), (5120, "serial", 3200, 1919, 1000),
    (5120, "side", 2560, 2560, 200), (5120, "side", 2597, 2522, 200),
    (6144, "serial", 3072, 3072, 257), (6144, "serial", 2561, 2560, 1500),
    (6144, "side", 3072, 3072, 64), (6144, "side", 3840, 2303, 64), (6144, "side", 2561, 2560, 200),
    (8192, "side", 4096, 4096, 64), (8192, "side", 4133, 4058, 64), (8192, "side", 3073, 3072, 150),
    (10240, "serial", 5120, 5120, 100), (10240, "serial", 6400, 3839, 100), (10240, "serial", 4097, 4096, 220),
    (12288, "serial", 6144, 6144, 64), (12288, "serial", 6181, 6106, 64), (12288, "serial", 5121, 5120, 100),
    (14336, "serial", 7168, 7168, 64), (14336, "serial", 8960, 5375, 64), (14336, "serial", 6145, 6144, 70),
    (16384, "serial", 8192, 8192, 64), (16384, "serial", 10240, 6143, 64), (16384, "serial", 7169, 7168, 64),
    (20480, "serial", 10240, 10240, 40), (20480, "serial", 10277, 10202, 40), (20480, "serial", 8193, 8192, 40),
    (24576, "serial", 12288, 12288, 40), (24576, "serial", 15360, 9215, 40), (24576, "serial", 10241, 10240, 40),
    (28672, "serial", 14336, 14336, 40), (28672, "serial", 14373, 14298, 40), (28672, "serial", 12289, 12288, 40),
    (32768, "serial", 16384, 16384, 40), (32768, "serial", 16421, 16346, 40), (32768, "serial", 14337, 14336, 40),
    (12288, "quarters", 6144, 6144, 5), (12288, "quarters", 7680, 4607, 5), (12288, "quarters", 5121, 5120, 5),
    (16384, "quarters", 8192, 8192, 5), (16384, "quarters", 10240, 6143, 5), (16384, "quarters", 7169, 7168, 5),
    (20480, "quarters", 10240, 10240, 5), (20480, "quarters", 10277, 10202, 5),
    (24576, "quarters", 12288, 12288, 5), (24576, "quarters", 15360, 9215, 5),
    (28672, "quarters", 14336, 14336, 5), (28672, "quarters", 12289, 12288, 5),
    (32768, "quarters", 16384, 16384, 5), (32768, "quarters", 16421, 16346, 5),
]

# products mod B^n: points, way, n, batch
LOW = [
    (2048, "side", 1024, 100), (2048, "side", 1023, 100),
    (3072, "side", 1536, 200), (3072, "side", 1535, 200), (3072, "side", 1351, 200),
    (4096, "side", 2048, 150), (4096, "side", 2047, 150), (4096, "side", 1793, 150),
    (8192, "side", 4096, 150), (8192, "side", 4095, 150), (8192, "side", 3585, 220),
    (10240, "serial", 5120, 1000), (10240, "serial", 5119, 1000),
    (12288, "serial", 6144, 200), (12288, "serial", 6143, 200), (12288, "serial", 5633, 512),
    (14336, "serial", 7168, 200), (14336, "serial", 6657, 220),
    (16384, "serial", 8192, 100), (16384, "serial", 8191, 100), (16384, "serial", 7169, 200),
    (20480, "serial", 10240, 70), (20480, "serial", 10239, 70), (20480, "serial", 8193, 220),
    (24576, "serial", 12288, 100), (24576, "serial", 12287, 100), (24576, "serial", 10241, 100),
    (28672, "serial", 14336, 70), (28672, "serial", 14335, 70), (28672, "serial", 12289, 70),
    (32768, "serial", 16384, 70), (32768, "serial", 16383, 70), (32768, "serial", 14337, 70),
    (12288, "quarters", 6143, 5), (16384, "quarters", 7681, 5), (20480, "quarters", 10239, 5),
    (24576, "quarters", 12287, 5), (28672, "quarters", 14335, 5), (32768, "quarters", 16383, 5),
]

GUARD = 67   # limbs on either side of a result (odd: results at odd limb addresses)


@pytest.fixture(scope="module")
def bi():
    import paper_2607_28897_amd as m
    m.lib()
    yield m
    m.set_mfma_config(0, 0, 0)


def operand(seed, batch, n, which):
    """[batch, n] limbs at an odd limb address, on the GPU, and the first rows."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randint(-2**31, 2**31, (batch * n + 1,), dtype=torch.int32, device="cuda", generator=g)
    x = x[1:].view(batch, n)
    x[0] = -1
    if which == "a":
        x[1] = -1
        x[2, :-1] = 0
        x[2, -1] = -1
        x[3, n // 2:] = -1                    # long runs against random limbs
    else:
        x[1, 1:] = 0
        x[1, 0] = 1                           # all ones, unchanged
        x[2] = -1
        x[3, : n // 3] = 0
    return x


def guarded(batch, n):
    import torch
    buf = torch.full((batch * n + 2 * GUARD,), 0x5a5a5a5a, dtype=torch.int32, device="cuda")
    return buf, buf[GUARD:-GUARD].view(batch, n)


def check(bi, orc, points, way, a, b, low):
    import torch
    L = bi.lib()
    (batch, na), nb = a.shape, b.shape[1]
    nout = na if low else na + nb
    quarters = way == "quarters"
    assert bi.mul_transform(na, nb, batch, low, quarters) == (points, way)
    s = torch.cuda.current_stream().cuda_stream
    size = ctypes.c_size_t()
    assert L.bigint_mul_workspace_size(na, nb, batch, ctypes.byref(size)) == 0
    # (a workspace is allocated to its last byte, with guards of its own)
    ws = torch.full((size.value + 256,), 0x5a, dtype=torch.uint8, device="cuda") if quarters else None
    args = (a.data_ptr(), b.data_ptr(), na) if low else (a.data_ptr(), na, b.data_ptr(), nb)
    tail = (batch,) if low else (batch, bi.MUL_AUTO)
    call = L.bigint_mullo if low else L.bigint_mul
    buf, out = guarded(batch, nout)
    if quarters:
        assert size.value > 0
        f = L.bigint_mullo_ws if low else L.bigint_mul_ws
        assert f(out.data_ptr(), *args, *tail, ws.data_ptr(), size.value, s) == 0
        assert bool((ws[size.value:] == 0x5a).all())
    else:
        assert call(out.data_ptr(), *args, *tail, s) == 0
    assert bool((buf[:GUARD] == 0x5a5a5a5a).all()) and bool((buf[-GUARD:] == 0x5a5a5a5a).all())
    want = torch.empty((batch, nout), dtype=torch.int32, device="cuda")
    bi.set_mfma_config(0, 8, 0)               # a forced configuration keeps the MFMA multiply
    assert bi.mul_transform(na, nb, batch, low, True) is None
    assert call(want.data_ptr(), *args, *tail, s) == 0
    bi.set_mfma_config(0, 0, 0)
    assert torch.nonzero((out != want).any(dim=1)).flatten().tolist() == []
    x, y, got = host(a[:4]), host(b[:4]), host(out[:4])
    exp = oracle_map(lambda i: (orc.mullo1 if low else orc.mul1)(x[i], y[i]), range(4))
    assert [i for i in range(4) if not np.array_equal(got[i], exp[i])] == []


@pytest.mark.parametrize("points,way,na,nb,batch", FULL)
def test_full(bi, orc, points, way, na, nb, batch):
    check(bi, orc, points, way, operand(na, batch, na, "a"), operand(nb + 1, batch, nb, "b"), False)


@pytest.mark.parametrize("points,way,n,batch", LOW)
def test_low(bi, orc, points, way, n, batch):
    check(bi, orc, points, way, operand(n, batch, n, "a"), operand(n + 1, batch, n, "b"), True)


@pytest.mark.parametrize("sizes,waves", [
    # leaf sizes 5..8 of 1024 and 512 threads, 5..8 and 2..4 side by side
    ([(10240, 10240), (12288, 12287), (14336, 14335), (16384, 16383), (8193, 8192), (16384, 2000)], 16),
    ([(5120, 5120), (6144, 6143), (7168, 7167), (8192, 8191), (4097, 4096), (8192, 2000)], 8),
    ([(2560, 2560), (3072, 3071), (3584, 3583), (4096, 4095), (2049, 2048), (4096, 1000)], 12),
    ([(1536, 1536), (2048, 2047), (2048, 2048), (1537, 1536), (1024, 1024)], 12),
])
def test_ragged_families(bi, sizes, waves):
    """One plan per kernel family: every leaf size, 1200 products in turn."""
    import torch
    n = [sizes[i % len(sizes)] for i in range(1200)]
    la, lb = (np.array([x[k] for x in n], np.int64) for k in range(2))
    off = [np.concatenate([[0], np.cumsum(x)]) for x in (la, lb, la + lb)]
    g = np.random.default_rng(len(sizes) + waves)
    a, b = (rand_limbs(g, int(o[-1])) for o in off[:2])
    a[: off[0][12]] = 0xFFFFFFFF
    b[: off[1][12]] = 0xFFFFFFFF
    ta, tb = (torch.from_numpy(x.view(np.int32)).cuda() for x in (a, b))
    oa, ob, oo = (torch.from_numpy(o).cuda() for o in off)
    plan = bi.MulPlan(la, lb)
    assert [s["waves"] for s in plan.segments()] == [waves] and plan.segments()[0]["instances"] == len(n)
    out, _ = plan(ta, oa, tb, ob, out_off=oo)
    # each size as a uniform batch of the MFMA-split multiply
    for k, (na, nb) in enumerate(sizes):
        rows = range(k, len(n), len(sizes))
        x = torch.stack([ta[off[0][i]:off[0][i + 1]] for i in rows])
        y = torch.stack([tb[off[1][i]:off[1][i + 1]] for i in rows])
        p = torch.stack([out[off[2][i]:off[2][i + 1]] for i in rows])
        assert bool((p == bi.mul(x, y, bi.MUL_MFMA)).all()), (na, nb)
    plan.close()
