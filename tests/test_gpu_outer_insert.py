"""R as a node of Q_1's product tree where the groups are kept (Alg. 2's form: a
product of prime powers from a factorisation, and C(n) one product per launch),
against R multiplied on after the tree: the same integer as the oracle's, with the
node really taken, or not."""
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


@pytest.mark.parametrize("fused", [None, 12])
@pytest.mark.parametrize("n", [5000, 100000, 262147, 1000003])
def test_product_of_groups(cat, n, fused):
    want = oracle.catalan(n)
    exps, off, primes = cat.factor(n)
    primes = primes.clone()
    try:
        cat.set_fused_levels(fused)
        for on in (True, False):
            cat.set_outer_node(on)
            for integer in (False, True):
                cat.set_integer_transforms(integer)
                print("product", n, "outer node", on, "fused", fused, "integer", integer, flush=True)
                assert np.array_equal(cat.to_numpy(cat.product(exps, off, primes)), want)
                lvl = cat.stats()["outer_level"]
                assert lvl >= 8 if on and n >= 262147 else on or lvl == -1, (on, lvl)
    finally:
        cat.set_integer_transforms(False)
        cat.set_outer_node(True)
        cat.set_fused_levels(None)


def test_plain_form(cat):
    n = 100000
    want = oracle.catalan(n)
    try:
        for on in (True, False):
            cat.set_outer_node(on)
            print("plain", n, "outer node", on, flush=True)
            assert np.array_equal(cat.to_numpy(cat.exact(n, mode="plain")), want)
            assert (cat.stats()["outer_level"] >= 6) == on
    finally:
        cat.set_outer_node(True)
