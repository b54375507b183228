"""CPU-only: the query of the transform that AUTO takes (256 CUs are assumed where
there is no GPU)."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def bi():
    import paper_2607_28897_amd as m
    if not os.path.exists(m.LIB_PATH):
        pytest.skip("library not built")
    m.lib()
    yield m
    m.set_mfma_config(0, 0, 0)


def test_arguments(bi):
    L, m, w = bi.lib(), ctypes.c_int(), ctypes.c_int()
    r = (ctypes.byref(m), ctypes.byref(w))
    assert L.bigint_mul_transform(4096, 4096, 64, 1, 0, *r) == 0
    assert L.bigint_mul_transform(4096, 4000, 64, 1, 0, *r) == bi.EINVAL   # mod B^n: one size
    assert L.bigint_mul_transform(0, 4096, 64, 0, 0, *r) == bi.EINVAL
    assert L.bigint_mul_transform(4096, 0, 64, 0, 0, *r) == bi.EINVAL
    assert L.bigint_mul_transform(4096, 4096, 0, 0, 0, *r) == bi.EINVAL
    assert L.bigint_mul_transform(4096, 4096, 64, 0, 0, None, r[1]) == bi.EINVAL
    assert L.bigint_mul_transform(4096, 4096, 64, 0, 0, r[0], None) == bi.EINVAL


def test_choice(bi):
    # the calls of perf/cases.py
    assert bi.mul_transform(1024, 1024, 64) is None
    assert bi.mul_transform(256, 256, 16384) is None
    assert bi.mul_transform(4096, 4096, 1024) == (8192, "side")
    assert bi.mul_transform(16384, 16384, 256) == (32768, "serial")
    assert bi.mul_transform(16384, 16384, 3) == (32768, "quarters")
    assert bi.mul_transform(5003, 2777, 300) == (8192, "side")
    assert bi.mul_transform(8192, 8192, 512, low=True) == (16384, "serial")
    # operands it does not take: short ones, more points than it has
    assert bi.mul_transform(16384, 63, 64) is None
    assert bi.mul_transform(16385, 16384, 64) is None
    # a forced configuration keeps the MFMA multiply
    bi.set_mfma_config(0, 8, 0)
    assert bi.mul_transform(16384, 16384, 256) is None
    bi.set_mfma_config(0, 0, 0)


@pytest.mark.parametrize("n", [4097, 6144, 8192, 10000, 16384])
@pytest.mark.parametrize("batch", [1, 40, 300, 5000])
def test_workspace_is_for_the_quarters(bi, n, batch):
    size = ctypes.c_size_t()
    assert bi.lib().bigint_mul_workspace_size(n, n, batch, ctypes.byref(size)) == 0
    t = bi.mul_transform(n, n, batch)
    assert (size.value > 0) == (t is not None and t[1] == "quarters")
    assert (bi.mul_transform(n, n, batch, workspace=False) or (0, ""))[1] != "quarters"


# measured without a workspace: us by the MFMA multiply, by transforms
@pytest.mark.parametrize("na,nb,batch,low,mfma,ntt", [
    (13000, 13000, 1, False, 92, 110), (12500, 12500, 8, False, 94, 111), (16384, 10922, 4, False, 91, 113),
    (16384, 5461, 8, False, 68, 82), (8192, 5461, 2, False, 50, 63), (9000, 9000, 1, False, 68, 73),
    (14000, 14000, 2, True, 89, 111), (14336, 14336, 10, True, 93, 111),
    (16384, 16384, 1, False, 113, 105), (10240, 10240, 4, False, 77, 72), (8192, 8192, 1, False, 62, 57),
    (4096, 4096, 8, False, 36, 24), (13000, 13000, 40, False, 306, 111), (14000, 14000, 20, True, 151, 111),
])
def test_few_products_without_workspace(bi, na, nb, batch, low, mfma, ntt):
    """So few that the MFMA multiply spreads each over the device: the faster one."""
    assert (bi.mul_transform(na, nb, batch, low, False) is None) == (mfma < ntt)


# us by the MFMA multiply, by transforms
@pytest.mark.parametrize("na,nb,batch,low,mfma,ntt", [
    (1700, 212, 257, False, 11.3, 17.8), (1300, 433, 257, False, 12.7, 17.7), (3000, 375, 300, False, 18.3, 23.8),
    (1536, 1024, 513, False, 24.5, 29.4), (2300, 766, 800, False, 33.1, 40.7), (1024, 1024, 257, True, 12.4, 17.3),
    (1024, 1024, 1024, False, 27.7, 33.2), (2048, 2048, 300, False, 34.2, 23.2), (1900, 1266, 400, False, 26.6, 23.2),
    (1536, 1536, 280, False, 25.2, 21.4), (2048, 2048, 280, True, 26.0, 22.5), (1900, 1900, 230, True, 16.8, 14.6),
    (1536, 1536, 256, True, 16.5, 13.6),
])
def test_rounds_of_small_transforms(bi, na, nb, batch, low, mfma, ntt):
    """Just above one or two products per CU the transforms take a round more."""
    assert (bi.mul_transform(na, nb, batch, low) is None) == (mfma < ntt)
