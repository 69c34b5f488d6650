"""Products and decimal text of stages whose outermost inverse pass recombines
the three primes itself (2^22 digits a batch and more): carries inside a run of
digits, out of it, through whole runs and across workgroups, at every column
length that takes this path, against closed forms and Python integers."""
import numpy as np
import pytest

from tests import pins

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cat():
    import torch

    import paper_2601_11621_amd as c

    torch.cuda.set_device(0)
    c.init(0)
    return c


def _ones_product(a, b):
    """(2^(32a) - 1) (2^(32b) - 1) as limbs."""
    x = (1 << 32 * (a + b)) - (1 << 32 * a) - (1 << 32 * b) + 1
    return np.frombuffer(x.to_bytes(4 * (a + b), "little"), dtype=np.uint32)


# 2^15 .. 2^19 digits: columns of 2^4 (twice) .. 2^7
@pytest.mark.parametrize("k", [15, 16, 17, 18, 19])
def test_batches(cat, k):
    rng = np.random.default_rng(k)
    cnt = (1 << (22 - k)) + 1
    n = 1 << k                                   # limbs of a full operand
    la = [n - int(d) for d in rng.integers(0, 200, cnt)]
    lb = [n - int(d) for d in rng.integers(0, 200, cnt)]
    la[0] = lb[0] = n
    la[1], lb[1] = n + 1, n                      # no coefficient at the top digit
    la[2], lb[2] = n - 1, n - 64                 # odd sums
    ops = []
    for i in range(cnt):
        if i % 4 == 3:                           # random against random
            x = rng.integers(0, 2**32, la[i], dtype=np.uint64).astype(np.uint32)
            y = rng.integers(0, 2**32, lb[i], dtype=np.uint64).astype(np.uint32)
        else:                                    # carries through every digit
            x = np.full(la[i], 0xFFFFFFFF, dtype=np.uint32)
            y = np.full(lb[i], 0xFFFFFFFF, dtype=np.uint32)
        if i % 8 == 4:                           # long zero and all-ones stretches
            y[:] = 0
            y[-1] = 1
        ops.append((x, y))
    a_off = np.concatenate([[0], np.cumsum(la)]).astype(np.uint64)
    b_off = np.concatenate([[0], np.cumsum(lb)]).astype(np.uint64)
    print("runs", k, cnt, flush=True)
    c, c_off = cat.mul_batched(cat.from_numpy(np.concatenate([x for x, _ in ops])), a_off,
                               cat.from_numpy(np.concatenate([y for _, y in ops])), b_off)
    c = cat.to_numpy(c)
    done = 0
    for i in range(cnt):
        got = c[int(c_off[i]):int(c_off[i]) + la[i] + lb[i]]
        if i % 8 == 4:
            want = np.concatenate([np.zeros(lb[i] - 1, np.uint32), ops[i][0], np.zeros(1, np.uint32)])
        elif i % 4 == 3:
            if k > 16 or done > 3:
                continue
            done += 1
            want = int.from_bytes(ops[i][0].tobytes(), "little") * int.from_bytes(ops[i][1].tobytes(), "little")
            want = np.frombuffer(want.to_bytes(4 * (la[i] + lb[i]), "little"), dtype=np.uint32)
        else:
            want = _ones_product(la[i], lb[i])
        assert np.array_equal(got, want), i


# 2^23 digits (the first prime set) and 2^24 (the second): two column passes, the
# second applying the first's twiddles
@pytest.mark.parametrize("la,lb", [(2**23, 2**23 - 3), (2**23 + 5, 2**23 + 64)])
def test_two_column_passes(cat, la, lb):
    print("two passes", la, lb, flush=True)
    a, b = (cat.from_numpy(np.full(n, 0xFFFFFFFF, dtype=np.uint32)) for n in (la, lb))
    c, _ = cat.mul_batched(a, [0, la], b, [0, lb])
    assert np.array_equal(cat.to_numpy(c)[:la + lb], _ones_product(la, lb))


@pytest.mark.parametrize("L,kind", [(8_000_003, "random"), (9_100_000, "ones")])
def test_decimal(cat, L, kind):
    x = np.full(L, 0xFFFFFFFF, dtype=np.uint32)
    if kind == "random":
        x = np.random.default_rng(L).integers(0, 2**32, L, dtype=np.uint64).astype(np.uint32)
    print("runs decimal", L, flush=True)
    text = cat.to_decimal_device(cat.from_numpy(x))
    s1, s2, g0 = pins.decimal_group_residues(text)
    assert s1 == pins.limbs_mod_vec(x, 10**9 - 1)
    assert s2 == pins.limbs_mod_vec(x, 10**9 + 1)
    assert g0 == pins.limbs_mod_vec(x, 10**9)
    assert text.numel() == cat.decimal_digits(cat.from_numpy(x))
