"""cat_outer_node_set between the two halves of an asynchronous request: the
ticket finishes in the form in which it was begun, and a later C(n) call of the
same n takes the form in force, bit for bit."""
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


@pytest.mark.parametrize("n", [5000, 100003])
@pytest.mark.parametrize("first", [True, False])
def test_switch_under_a_ticket(cat, n, first):
    import torch

    lib = cat.load()
    want = oracle.catalan(n)
    _, max_limbs, wbytes = cat.sizes(n)
    w = torch.empty(wbytes, dtype=torch.uint8, device="cuda")
    out = torch.empty(max_limbs, dtype=torch.int32, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    t, nl = ctypes.c_void_p(), ctypes.c_size_t()
    try:
        cat.set_outer_node(first)
        cat._check(lib.catalan_begin(n, cat._ptr(w), wbytes, st, ctypes.byref(t)), "catalan_begin")
        while lib.cat_ticket_query(t) == cat.CAT_EAGAIN:
            pass
        cat.set_outer_node(not first)
        cat._check(lib.catalan_continue(t, cat._ptr(out), max_limbs), "catalan_continue")
        cat._check(lib.catalan_end(t, ctypes.byref(nl)), "catalan_end")
        assert np.array_equal(cat.to_numpy(out[:nl.value]), want)
        for k in range(3):   # (the switch stays: setting it again would drop the plans)
            print("n", n, "outer node", not first, "call", k, flush=True)
            assert np.array_equal(cat.to_numpy(cat.exact(n)), want), k
    finally:
        cat.set_outer_node(True)
