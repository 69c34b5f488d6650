"""The bottom of the product trees (nodes of 256 limbs, as many entries per eight
limbs as their bit length allows) and the powers form of C(n): exact against
Python's integers and the oracle."""
import math

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


@pytest.mark.parametrize("bits", [1, 2, 10, 11, 16, 21, 25, 28, 31, 32])
def test_entries_per_node(cat, bits):
    """Entry counts around a piece (s entries per eight limbs), a node (32 s) and
    two nodes, all entries of the full bit length (the fullest pieces) or random
    below it, in one group or split over two exponents."""
    s = min(256 // bits, 24)
    rng = np.random.default_rng(bits)
    for k in sorted({1, 2, s - 1, s, s + 1, 7 * s + 1, 32 * s - 1, 32 * s, 32 * s + 1, 64 * s, 65 * s + 3, 257} - {0}):
        for kind in ("full", "rand"):
            top = (1 << bits) - 1
            e = np.full(k, top, dtype=np.uint64) if kind == "full" else rng.integers(1, top + 1, k, dtype=np.uint64)
            e = e.astype(np.uint32)
            print("bits", bits, "entries", k, kind, flush=True)
            got = cat.to_int(cat.product([1], [0, k], e))
            assert got == math.prod(int(x) for x in e), (bits, k, kind)
            cut = k // 2
            if cut:
                got = cat.to_int(cat.product([1, 3], [0, cut, k], e))
                want = math.prod(int(x) for x in e[:cut]) * math.prod(int(x) for x in e[cut:]) ** 3
                assert got == want, (bits, k, kind, cut)


def test_longer_entries_than_announced(cat):
    """An entry longer than max_entry_bits, among shorter ones that keep the sum
    within bounds, was always multiplied correctly."""
    e = np.array([2**31 - 1] + [3] * 40, dtype=np.uint32)
    assert cat.to_int(cat.product([1], [0, 41], e, max_entry_bits=8)) == (2**31 - 1) * 3**40


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 30, 31, 1 << 10, (1 << 14) - 1, 1 << 14, (1 << 17) + 1, 1 << 20])
def test_powers_form(cat, n):
    """C(n) as one product of prime powers, at changes of the entries' bit length
    (2n a power of two) and where R becomes a node of its own, in every mode, as
    a batch of requests, and with R kept out of the tree."""
    want = oracle.catalan(n)
    for mode in ["graph", "batched"] + (["plain"] if n < 2000 else []):
        assert np.array_equal(cat.to_numpy(cat.exact(n, mode=mode)), want), (n, mode)
    for x in cat.exact_batch([n, n, 5, n + 1])[:2]:
        assert np.array_equal(cat.to_numpy(x), want), n
    try:
        cat.set_outer_node(False)
        assert np.array_equal(cat.to_numpy(cat.exact(n)), want), n
    finally:
        cat.set_outer_node(True)
