"""Factorial ratios of the smallest arguments: below 4 the square root of the
largest one is below 2, which the sieve of odd numbers does not hold."""
import itertools
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


@pytest.mark.parametrize("top", range(0, 10))
def test_one_over_one_or_two(cat, top):
    for k in range(0, 3):
        for den in itertools.combinations_with_replacement(range(0, top + 1), k):
            q, r = divmod(math.factorial(top), math.prod(math.factorial(d) for d in den))
            if r:
                with pytest.raises(cat.CatalanError):
                    cat.ratio_exact([top], den)
                continue
            for mode in ("batched", "plain"):
                assert cat.to_int(cat.ratio_exact([top], den, mode=mode)) == q, (top, den, mode)
            assert np.array_equal(cat.to_numpy(cat.ratio_exact([top], den)), oracle.ratio([top], list(den)))


def test_factors(cat):
    """{2: 1} and {2: 1, 3: 1}, by exponent bits."""
    for num, want in (([2], [2]), ([3], [2, 3]), ([2, 2], [2])):
        exps, off, primes = cat.ratio_factor(num, [])
        assert cat.to_numpy(primes).tolist() == want, num
        assert exps.tolist() == ([2] if len(num) == 2 else [1])
