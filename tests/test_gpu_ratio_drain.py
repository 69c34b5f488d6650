"""factorial_ratio_exact synchronises: a call that ends in an error has no launch
of its own left in the caller's workspace, whichever step found the error."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cat():
    import torch

    import paper_2601_11621_amd as c

    torch.cuda.set_device(0)
    c.init(0)
    return c


def test_no_work_in_flight_after_an_error(cat):
    """N = A! / A! = 1 without room for its limb (the plan finds that out, while
    the last kernel of Phase 1 covers 30,518 segments)."""
    import torch

    lib = cat.load()
    A = 10**9
    arr = (ctypes.c_uint64 * 1)(A)
    p, q, wb = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t()
    cat._check(lib.factorial_ratio_sizes(arr, 1, arr, 1, ctypes.byref(p), ctypes.byref(q), ctypes.byref(wb)), "sizes")
    work = torch.empty(wb.value, dtype=torch.uint8, device="cuda")
    out = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    nl = ctypes.c_size_t()
    for k in range(3):
        print("call", k, flush=True)
        r = lib.factorial_ratio_exact(arr, 1, arr, 1, cat._ptr(out), 0, ctypes.byref(nl), cat._ptr(work), wb.value,
                                      ctypes.c_void_p(st.cuda_stream), 0)
        idle = st.query()
        torch.cuda.synchronize()
        assert r == cat.CAT_ERANGE and nl.value == 1
        assert idle, k
    assert out.tolist() == [-1] * 4
