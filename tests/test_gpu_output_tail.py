"""What lies behind the result in the caller's buffer: the calls that return C(n)
without a graph write its limbs and nothing else; so does the first call that
would use one."""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cat():
    import torch

    import paper_2601_11621_amd as c

    torch.cuda.set_device(0)
    c.init(0)
    return c


NS = [0, 1, 2, 13, 16, 17, 18, 19, 33, 100, 1000, 4097, 99991, 250007, 1000003]


@pytest.mark.parametrize("call,n", [(c, n) for c in ("noalloc", "batched", "plain", "first") for n in NS
                                    if c != "plain" or n <= 10**5])   # (a launch per product)
def test_nothing_behind_the_result(cat, call, n):
    import torch

    lib = cat.load()
    want = oracle.catalan(n)
    _, max_limbs, wbytes = cat.sizes(n)
    cap = max(max_limbs, len(want)) + 4096
    w = torch.empty(wbytes, dtype=torch.uint8, device="cuda")
    out = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    nl = ctypes.c_size_t()
    print(call, n, flush=True)
    if call == "noalloc":
        r = lib.catalan_exact_noalloc(n, cat._ptr(out), cap, ctypes.byref(nl), st)
    else:
        cat.set_outer_node(True)   # (drops the plans: the call is the first for n)
        flags = {"batched": 0, "plain": 1, "first": 2}[call]
        r = lib.catalan_exact_ex(n, cat._ptr(out), cap, ctypes.byref(nl), cat._ptr(w), wbytes, st, flags)
    assert r == cat.CAT_OK and nl.value == len(want)
    got = cat.to_numpy(out)
    assert np.array_equal(got[:nl.value], want)
    assert (got[nl.value:] == 0xFFFFFFFF).all()
