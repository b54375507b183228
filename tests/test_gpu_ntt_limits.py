"""Batches of the transform multiply at the limit of one launch (fewer than
2^32 work-items, 5,592,405 work-groups of 768 threads): the products on both
sides of the boundary and a sample of the others against the oracle.  Operands
of 1760 limbs are the smallest that the side-by-side kernels take in such
batches; 119 GB of device memory."""
import numpy as np
import pytest

from gpu_util import host, oracle_map

pytestmark = pytest.mark.gpu

N, GROUPS = 1760, (2**32 - 1) // 768
BATCH = GROUPS + 7


@pytest.fixture(scope="module")
def operands():
    import torch
    need = 3 * N * BATCH * 4 + (4 << 30)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip(f"needs {need >> 30} GiB of free device memory")
    g = torch.Generator(device="cuda").manual_seed(2607)
    a = torch.randint(-2**31, 2**31, (BATCH, N), dtype=torch.int32, device="cuda", generator=g)
    yield a
    del a
    torch.cuda.empty_cache()


def check(orc, a, p):
    rows = sorted({0, 1, GROUPS - 1, GROUPS, GROUPS + 1, BATCH - 1} | set(range(17, BATCH, BATCH // 20)))
    assert len(rows) >= 20
    x, got = host(a[rows]), host(p[rows])
    want = oracle_map(lambda i: orc.mul1(x[i], x[i]), range(len(rows)))
    assert [r for i, r in enumerate(rows) if not np.array_equal(got[i], want[i])] == []


@pytest.mark.timeout(170)
def test_uniform(orc, operands):
    import paper_2607_28897_amd as bi
    a = operands
    check(orc, a, bi.mul(a, a))


@pytest.mark.timeout(170)
def test_ragged(orc, operands):
    import torch
    import paper_2607_28897_amd as bi
    a = operands
    n = np.full(BATCH, N, np.int64)
    off = torch.arange(0, (BATCH + 1) * N, N, dtype=torch.int64, device="cuda")
    plan = bi.MulPlan(n, n, bi.PLAN_NO_GRAPH)
    assert plan.segments()[0]["waves"] == 12          # the side-by-side transforms
    p, _ = plan(a.view(-1), off, a.view(-1), off, out_off=2 * off)
    check(orc, a, p.view(BATCH, 2 * N))
    plan.close()
