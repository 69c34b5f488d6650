"""The four-step FP64 transforms, one case per transform length: every length of a
column pass (2^4 .. 2^10 digits in one pass, 2^5 .. 2^7 in two), rows of 2^11 and
2^12, both prime sets, one product and several, operands of both halves and of
the lower half only.  Exact: all-ones products against their closed form, others
by residues modulo 2^32 - 5, 2^32 + 1 and 2^32 - 1."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MODULI = [2**32 - 5, 2**32 + 1, 2**32 - 1]


@pytest.fixture(scope="module")
def cat():
    import torch

    import paper_2601_11621_amd as c

    torch.cuda.set_device(0)
    c.init(0)
    return c


def _ones_product(a, b):
    """(2^(32a) - 1) (2^(32b) - 1) as limbs, a >= b: 1, zeros, 2^32 - 2 or ones from
    limb b on, 2^32 - 2 at limb a, ones above."""
    c = np.zeros(a + b, dtype=np.uint32)
    c[0] = 1
    if a == b:
        c[a] = 0xFFFFFFFE
        c[a + 1:] = 0xFFFFFFFF
    else:
        c[b:a] = 0xFFFFFFFF
        c[a] = 0xFFFFFFFE
        c[a + 1:] = 0xFFFFFFFF
    return c


def test_closed_form():
    for a, b in [(1, 1), (2, 1), (5, 5), (7, 3)]:
        x = (2**(32 * a) - 1) * (2**(32 * b) - 1)
        assert int.from_bytes(_ones_product(a, b).astype("<u4").tobytes(), "little") == x


@pytest.mark.parametrize("logd", range(15, 26))
def test_transform_length(cat, logd):
    rng = np.random.default_rng(logd)
    n = 1 << (logd + 1)                       # limbs of the transform
    # the product fills the transform or just needs it; one operand beyond its half
    shapes = [(n // 2, n // 2, "ones"), (n // 2 + 1, n // 2, "ones"), (n - n // 8, n // 8, "ones"),
              (n // 4 + 5, n // 4 + 3, "rand"), (n - 2000, 1999, "rand"), (n // 2 - 3, n // 2 - 64, "rand")]
    if logd >= 23:
        shapes = [shapes[1], shapes[3]]
    for count in ((1, 3) if logd <= 21 else (1,)):
        for la, lb, kind in shapes:
            print("digits 2^%d" % logd, count, "x", la, lb, kind, flush=True)
            a, b = (np.full(m * count, 0xFFFFFFFF, dtype=np.uint32) if kind == "ones" else
                    rng.integers(0, 2**32, m * count, dtype=np.uint64).astype(np.uint32) for m in (la, lb))
            da, db = cat.from_numpy(a), cat.from_numpy(b)
            off = [m * np.arange(count + 1, dtype=np.uint64) for m in (la, lb)]
            cat.timer_set("k_frow")
            try:
                c, _ = cat.mul_batched(da, off[0], db, off[1])
                assert cat.timer_get()[1] == 1, "not one four-step launch"
            finally:
                cat.timer_set(None)
            for i in range(count):
                x, y = da[la * i:la * (i + 1)], db[lb * i:lb * (i + 1)]
                z = c[(la + lb) * i:(la + lb) * (i + 1)]
                if kind == "ones":
                    assert np.array_equal(cat.to_numpy(z), _ones_product(la, lb)), i
                else:
                    r = [cat.residues(v) for v in (x, y, z)]
                    assert [p * q % m for p, q, m in zip(r[0], r[1], MODULI)] == list(r[2]), i
