"""Scratch that the integer transforms needed and that stays enough: the 64-bit
digits of the FP64 transforms ask for no larger workspace, so every n that fitted
a given scratch still fits it.  Host-only size queries."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def cat():
    import paper_2601_11621_amd as c

    c.load()
    return c


# bytes asked for with one 32-bit limb per coefficient
@pytest.mark.parametrize("n,most", [(0, 5469696), (1, 5469696), (10, 5472000), (1000, 5981184), (10**5, 9691904),
                                    (10**6, 24362496), (10**7, 148626944), (10659042, 150993920),
                                    (10659142, 150993920), (10**8, 1148248576), (2050572903, 18652893184),
                                    (2147483647, 18910063616)])
def test_catalan(cat, n, most):
    assert cat.sizes(n)[2] <= most


def test_largest_n_without_allocation(cat):
    assert cat.sizes(10659142)[2] <= cat.noalloc_max_bytes()
    assert cat.sizes(10659143)[2] > cat.noalloc_max_bytes()


@pytest.mark.parametrize("num,den,most", [([64], [32, 32], 5257216), ([2 * 10**7], [10**7, 10**7], 362107136),
                                          ([10**6], [], 160907520), ([10**9], [10**9], 17264969216),
                                          ([77], [77], 5256960), ([10**8], [5 * 10**7, 5 * 10**7], 1518152192)])
def test_ratio(cat, num, den, most):
    assert cat.ratio_sizes(num, den)[2] <= most


@pytest.mark.parametrize("exps,off,bits,most", [([1], [0, 1], 32, 5252352), ([1], [0, 1000], 25, 5296640),
                                                ([1, 2], [0, 10**6, 10**6 + 300], 26, 157087488),
                                                ([1], [0, 1857859], 26, 303038208)])
def test_product(cat, exps, off, bits, most):
    lib = cat.load()
    e = (ctypes.c_uint32 * len(exps))(*exps)
    o = (ctypes.c_uint64 * len(off))(*off)
    ml, wb = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.prime_power_product_sizes(e, o, len(exps), bits, ctypes.byref(ml), ctypes.byref(wb)) == cat.CAT_OK
    assert wb.value <= most


@pytest.mark.parametrize("ns,most", [([1000], 5881856), ([1000, 10**7], 145528576),
                                     ([1000 * 2**i for i in range(14)], 282715904), ([10**6] * 32, 582960896)])
def test_batch(cat, ns, most):
    lib = cat.load()
    a = (ctypes.c_uint64 * len(ns))(*ns)
    wb = ctypes.c_size_t()
    assert lib.catalan_batch_sizes(len(ns), a, ctypes.byref(wb)) == cat.CAT_OK
    assert wb.value <= most


@pytest.mark.gpu
def test_largest_n_without_allocation_runs(cat):
    import torch

    n = 10659142
    cat.init(0)
    ref = cat.exact(n)
    out = torch.empty_like(ref)
    nl = ctypes.c_size_t()
    print("noalloc", n, flush=True)
    st = cat.load().catalan_exact_noalloc(n, cat._ptr(out), out.numel(), ctypes.byref(nl),
                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == cat.CAT_OK and nl.value == ref.numel() and torch.equal(out, ref)
