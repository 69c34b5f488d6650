"""The integer transforms (cat_integer_transforms_set): every prime set, and the
tiles, rows and column passes that the schedule table can ask of them, bit for
bit against the FP64 transforms and the oracle; the kernel timer says that the
kernels meant are the ones that run."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _rand, _schedule_rows11, _schedule_short, _schedule_tiles14, _schedule_wide

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cat():
    import torch

    import paper_2601_11621_amd as c

    torch.cuda.set_device(0)
    c.init(0)
    return c


def _batch(cat, seed):
    """Products of 2^4 .. 2^15 limbs and transforms of 2^17 .. 2^20 points."""
    rng = np.random.default_rng(seed)
    la = np.rint(2 ** rng.uniform(4, 15, 40)).astype(np.int64).tolist() + [1 << 16, (1 << 18) - 5, 300000, 600000]
    lb = np.rint(2 ** rng.uniform(4, 15, 40)).astype(np.int64).tolist() + [1 << 16, (1 << 18) - 3, 70000, 400000]
    a = np.concatenate([_rand(rng, n, "ones" if i % 3 == 0 else "rand") for i, n in enumerate(la)])
    b = np.concatenate([_rand(rng, n, "ones" if i % 3 == 0 else "rand") for i, n in enumerate(lb)])
    off = [np.concatenate([[0], np.cumsum(x)]).astype(np.uint64) for x in (la, lb)]
    return cat.from_numpy(a), off[0], cat.from_numpy(b), off[1]


def _launches(cat, kernel, f):
    cat.timer_set(kernel)
    try:
        r = f()
        return r, cat.timer_get()[1]
    finally:
        cat.timer_set(None)


@pytest.mark.parametrize("lazy", [0, 18, 22, 23])
@pytest.mark.parametrize("schedule", [None, _schedule_short, _schedule_wide, _schedule_rows11, _schedule_tiles14],
                         ids=["default", "short", "wide", "rows11", "tiles14"])
def test_schedules(cat, schedule, lazy):
    import torch

    base = cat.get_tuning()
    args = _batch(cat, 11)
    c0, _ = cat.mul_batched(*args)
    c0 = c0.clone()
    want = {n: oracle.catalan(n) for n in (5000, 100000)}
    t = cat.get_tuning()
    if schedule:
        schedule(t)
    try:
        cat.set_lazy_primes(lazy)
        cat.set_integer_transforms(True)
        cat.set_tuning(t)
        print("schedule", schedule and schedule.__name__, "lazy", lazy, flush=True)
        for kernel, some in [("k_row", True), ("k_frow", False), ("k_fcrt", False), ("k_crt", True)]:
            (c1, _), count = _launches(cat, kernel, lambda: cat.mul_batched(*args))
            assert (count > 0) == some, kernel
            assert torch.equal(c0, c1), kernel
        for n, x in want.items():
            for mode in ("batched", "graph", "graph"):
                assert np.array_equal(cat.to_numpy(cat.exact(n, mode=mode)), x), (n, mode)
    finally:
        cat.set_tuning(base)
        cat.set_integer_transforms(False)
        cat.set_lazy_primes(23)
    (c1, _), count = _launches(cat, "k_frow", lambda: cat.mul_batched(*args))
    assert count > 0 and torch.equal(c0, c1)


@pytest.mark.parametrize("lazy", [0, 22, 23])
@pytest.mark.parametrize("k", [21, 22, 23, 24])
def test_longest_of_each_prime_set(cat, k, lazy):
    """All-ones and random operands around 2^(k-1) limbs: the largest coefficients
    that a set has to hold, at the last sizes of the primes below 2^30."""
    import torch

    rng = np.random.default_rng(k)
    n = 1 << (k - 1)
    for la, lb, kind in [(n, n, "ones"), (n - 7, n // 3, "rand")]:
        a, b = cat.from_numpy(_rand(rng, la, kind)), cat.from_numpy(_rand(rng, lb, kind))
        c0 = cat.mul_batched(a, [0, la], b, [0, lb])[0].clone()
        try:
            cat.set_lazy_primes(lazy)
            cat.set_integer_transforms(True)
            print("2^%d points" % k, "lazy", lazy, kind, flush=True)
            c1, _ = cat.mul_batched(a, [0, la], b, [0, lb])
            assert torch.equal(c0, c1), (la, lb, kind)
        finally:
            cat.set_integer_transforms(False)
            cat.set_lazy_primes(23)


def test_switch_limits(cat):
    assert cat.load().cat_integer_transforms_set(2) == cat.CAT_EINVAL
