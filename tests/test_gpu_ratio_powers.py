"""Factorial ratios whose value comes from one tree of prime powers (every
p^v_p(N) as short as the largest argument) against those that need the groups
by exponent bits, at the edges between the two, bit for bit against the
oracle."""
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


@pytest.mark.parametrize("num,den", [
    ([64], [32, 32]), ([64], [1, 63]), ([2**16], [1, 2**16 - 1]), ([2**16 + 1], [2, 2**16 - 1]), ([77], [77]),
    # 2^v_2 one bit longer than the largest argument, and as long as it
    ([4], [1, 1, 1, 1]), ([4], [2, 1, 1]), ([4], [2, 2]), ([31], [16, 8, 4, 2, 1]), ([31], [15, 8, 4, 2, 1, 1]),
    # a large prime squared: 101^2 in 202! / 100!^2
    ([202], [100, 100]), ([70000], [35000, 34999, 1]), ([65537, 65537], [65536, 65536]),
    ([300000], [150000, 150000]), ([300000], [100000, 100000, 100000]),
])
def test_powers_and_groups(cat, num, den):
    print("ratio", num, den, flush=True)
    assert np.array_equal(cat.to_numpy(cat.ratio_exact(num, den)), oracle.ratio(num, den))
