"""GPU parity of the transform multiply (bigint_mul AUTO and bigint_mullo pick
it): at the edges of its transform sizes (M = 4 q T points), on operands of
all ones (the largest coefficients, carries through every block), zeros and
single limbs, against the MFMA-split multiply on every instance and the oracle
on the first rows; integers throughout, so the bytes are equal."""
import numpy as np
import pytest

from gpu_util import dev, host, oracle_map, rand_limbs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bi():
    import paper_2607_28897_amd as m
    m.lib()
    yield m
    m.set_mfma_config(0, 0, 0)


def operands(seed, batch, na, nb):
    g = np.random.default_rng(100000 + seed)
    a, b = rand_limbs(g, batch, na), rand_limbs(g, batch, nb)
    a[0], b[0] = 0xFFFFFFFF, 0xFFFFFFFF
    a[1], b[1] = 0xFFFFFFFF, 0
    b[1, 0] = 1                                   # all ones, unchanged
    a[2] = 0
    a[2, -1] = 0xFFFFFFFF
    b[2] = 0xFFFFFFFF
    a[3, na // 2:] = 0xFFFFFFFF                   # long runs against random limbs
    b[3, : nb // 3] = 0
    return a, b


# every transform size: the largest operands that fit, one limb more (the next
# size), odd and unequal ones
EDGES = [(64, 640), (64, 768), (64, 896), (64, 1024), (128, 1280), (128, 1536), (128, 1792), (128, 2048),
         (256, 2560), (256, 3072), (256, 3584), (256, 4096), (512, 5120), (512, 6144), (512, 7168),
         (512, 8192), (1024, 10240), (1024, 12288), (1024, 14336), (1024, 16384)]


@pytest.mark.parametrize("T,n", EDGES)
@pytest.mark.parametrize("da,db", [(0, 0), (-1, 0), (1, 0), (-3, -200)])
def test_full_products(bi, orc, T, n, da, db):
    na, nb = n + da, n + db
    if na + nb > 32768:
        na = 16384
    batch = max(5, 4096 * 64 // T) if T < 256 else 5
    a, b = operands(n + da + 5 * db, batch, na, nb)
    ta, tb = dev(a), dev(b)
    p = bi.mul(ta, tb)
    want = bi.mul(ta, tb, bi.MUL_MFMA)
    assert bool((p == want).all())
    exp = oracle_map(lambda i: orc.mul1(a[i], b[i]), range(4))
    got = host(p[:4])
    assert all(np.array_equal(got[i], exp[i]) for i in range(4))


@pytest.mark.parametrize("na,nb,batch", [(1280, 1280, 2048), (1536, 1535, 2500), (2560, 2560, 1024), (3072, 3071, 900),
                                         (2561, 2561, 1024), (1024, 1025, 4096)])
def test_large_batches(bi, na, nb, batch):
    """The sizes whose large batches run one prime after another and whose
    small ones run the primes side by side: the same bytes."""
    a, b = operands(na * 3 + nb, batch, na, nb)
    ta, tb = dev(a), dev(b)
    p = bi.mul(ta, tb)
    assert bool((p == bi.mul(ta, tb, bi.MUL_MFMA)).all())
    assert bool((p[:9] == bi.mul(ta[:9].contiguous(), tb[:9].contiguous())).all())


@pytest.mark.parametrize("n,batch", [(2048, 2048), (2559, 6), (4096, 5), (5000, 5), (8192, 5), (9999, 4),
                                     (16383, 4), (16384, 5)])
def test_products_mod_bn(bi, orc, n, batch):
    a, b = operands(n, batch, n, n)
    ta, tb = dev(a), dev(b)
    p = bi.mullo(ta, tb)
    bi.set_mfma_config(0, 8, 0)                   # a forced configuration keeps the MFMA multiply
    want = bi.mullo(ta, tb)
    bi.set_mfma_config(0, 0, 0)
    assert bool((p == want).all())
    got = host(p[:4])
    assert all(np.array_equal(got[i], orc.mul1(a[i], b[i])[:n]) for i in range(4))


@pytest.mark.parametrize("na,nb", [(16384, 5000), (12000, 2500), (7000, 16384)])
def test_unequal_operands(bi, orc, na, nb):
    a, b = operands(na + nb, 4, na, nb)
    p = bi.mul(dev(a), dev(b))
    exp = oracle_map(lambda i: orc.mul1(a[i], b[i]), range(4))
    got = host(p)
    assert all(np.array_equal(got[i], exp[i]) for i in range(4))


@pytest.mark.parametrize("flags", [0, 2])
def test_ragged_unequal(bi, flags):
    """A plan over every transform family and leaf size, operands of unequal
    lengths at odd offsets, against the plain kernel's plan; graph replays and
    direct launches."""
    import torch
    g = np.random.default_rng(17)
    la = np.exp(g.uniform(np.log(600), np.log(16384), 700)).astype(np.int64)
    lb = np.maximum(64, (la * g.uniform(0.5, 1.0, 700)).astype(np.int64))
    edges = [1024, 1536, 2048, 2560, 3072, 3584, 4096, 5120, 6144, 7168, 8192, 10240, 12288, 14336, 16384]
    for k, n in enumerate(edges):
        la[2 * k:2 * k + 2] = n
        lb[2 * k:2 * k + 2] = [n, n - 1]
    off = [np.zeros(701, np.int64) for _ in range(2)]
    for o, n in zip(off, (la, lb)):
        np.cumsum(n, out=o[1:])
    a, b = (rand_limbs(g, int(o[-1])) for o in off)
    a[: off[0][20]] = 0xFFFFFFFF
    b[: off[1][20]] = 0xFFFFFFFF
    ta, tb = dev(a), dev(b)
    oa, ob = (torch.from_numpy(o).cuda() for o in off)
    plan, plain = bi.MulPlan(la, lb, flags), bi.MulPlan(la, lb, bi.PLAN_PLAIN)
    assert len(plan.segments()) >= 4
    want, oo = plain(ta, oa, tb, ob)
    out = torch.empty_like(want)
    for _ in range(3):
        out.fill_(-1)
        plan(ta, oa, tb, ob, out=out, out_off=oo)
        assert bool((out == want).all())
    plan.close()
    plain.close()


def test_graph_capture(bi):
    """A call with no workspace: captured and replayed, eager work between."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    a = torch.randint(-2**31, 2**31, (8, 4096), dtype=torch.int32, device="cuda", generator=g)
    b = torch.randint(-2**31, 2**31, (8, 4096), dtype=torch.int32, device="cuda", generator=g)
    want = bi.mul(a, b, bi.MUL_MFMA)
    bi.mul(a, b)
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr):
        p = bi.mul(a, b)
    for _ in range(3):
        p.zero_()
        gr.replay()
        torch.cuda.synchronize()
        assert bool((p == want).all())
        bi.add(a, b)


@pytest.mark.parametrize("na,nb", [(4097, 4096), (6144, 6144), (6145, 6144), (8192, 8192), (8193, 8192), (10240, 10240),
                                   (12288, 12287), (14336, 14336), (16384, 16384), (16384, 256), (16000, 4000),
                                   (9000, 700)])
def test_few_large_products(bi, orc, na, nb):
    """Few large products, every prime and quarter of each its own work-group:
    every transform size, unequal operands (one run of limbs only), all-ones
    and zero operands (carries through whole strips)."""
    a, b = operands(na + 2 * nb, 5, na, nb)
    p = bi.mul(dev(a), dev(b))
    exp = oracle_map(lambda i: orc.mul1(a[i], b[i]), range(5))
    got = host(p)
    assert [i for i in range(5) if not np.array_equal(got[i], exp[i])] == []
    if na == nb:
        got = host(bi.mullo(dev(a), dev(b)))
        assert [i for i in range(5) if not np.array_equal(got[i], exp[i][:na])] == []


def test_few_large_products_in_chunks(bi):
    """More products than share the workspace at once, and the C entry with a
    workspace too small for them (which then uses none)."""
    import ctypes
    import torch
    L = bi.lib()
    a, b = operands(9, 300, 10000, 9000)
    ta, tb = dev(a), dev(b)
    want = bi.mul(ta, tb, bi.MUL_MFMA)
    size = ctypes.c_size_t()
    assert L.bigint_mul_workspace_size(10000, 9000, 300, ctypes.byref(size)) == 0 and size.value > 0
    assert bool((bi.mul(ta, tb) == want).all())
    ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(want)
    args = (out.data_ptr(), ta.data_ptr(), 10000, tb.data_ptr(), 9000, 300, bi.MUL_AUTO, ws.data_ptr())
    s = torch.cuda.current_stream().cuda_stream
    assert L.bigint_mul_ws(*args, size.value // 2, s) == 0
    assert bool((out == want).all())
    assert L.bigint_mul_ws(out.data_ptr(), ta.data_ptr(), 10000, tb.data_ptr(), 9000, 300, bi.MUL_AUTO,
                           out.data_ptr(), 1 << 20, s) == bi.EINVAL
