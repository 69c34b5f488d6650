"""Decimal text at the edges of the conversion's levels: leaves of 29 limbs and
nodes of 29 2^j, one limb to either side (a last node of one limb, carried up
or joined), against the oracle's schoolbook division, character for character."""
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


# 29 2^j for the products inside one workgroup with carries (2^5 .. 2^11
# digits: j <= 6), without (up to 2^14: j <= 9) and over several (j >= 10)
@pytest.mark.parametrize("nodes", [1, 2, 3, 5, 8, 21, 64, 127, 128, 129, 512, 1024, 1025])
@pytest.mark.parametrize("d", [-1, 0, 1])
def test_node_edges(cat, nodes, d):
    L = 29 * nodes + d
    print("decimal node edge", L, flush=True)
    x = np.random.default_rng(L).integers(0, 2**32, size=L, dtype=np.uint64).astype(np.uint32)
    assert cat.to_decimal(cat.from_numpy(x)) == oracle.to_decimal(x)
    # zeros below one high limb: every addend zero, digits of powers of two
    x[:-1] = 0
    assert cat.to_decimal(cat.from_numpy(x)) == oracle.to_decimal(x)
    x[:] = 0xFFFFFFFF
    assert cat.to_decimal(cat.from_numpy(x)) == oracle.to_decimal(x)
