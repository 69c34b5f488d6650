"""Batches with more exponent groups than one plan holds (32), which run as
several plans one after another in one workspace: with the outer node off a
request brings a group per exponent, and eight of mixed sizes fill two plans.
Every result against the oracle, bit for bit."""
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


@pytest.mark.parametrize("ns", [
    # small requests first, so that the plans after the first write more than
    # the first one's results take
    [1000, 3727, 13894, 51794, 77777, 193069, 300000, 500000, 719685, 1000000],
    [1000000, 1000, 0, 300000, 5, 1, 20000, 77777, 4000, 500000, 193069, 3727],
    [30 + 7 * i for i in range(30)] + [200000, 1],
], ids=["ascending", "mixed", "many"])
def test_several_plans(cat, ns):
    want = {n: oracle.catalan(n) for n in ns}
    try:
        cat.set_outer_node(False)
        groups = sum(len(cat.factor(n)[0]) for n in ns)
        print("batch of", len(ns), "requests,", groups, "groups", flush=True)
        assert groups > 32
        for _ in range(2):
            for n, x in zip(ns, cat.exact_batch(ns)):
                assert np.array_equal(cat.to_numpy(x), want[n]), n
    finally:
        cat.set_outer_node(True)
    for n, x in zip(ns, cat.exact_batch(ns)):
        assert np.array_equal(cat.to_numpy(x), want[n]), n
