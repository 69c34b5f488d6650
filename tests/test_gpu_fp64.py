"""The FP64 transforms at the edges of their digits, tiles, rows and column
passes: exact against Python's integers, or by three residues of the product
where those would take long.  All arithmetic is exact, so the tolerance is
zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cat():
    import torch

    import paper_2601_11621_amd as c

    torch.cuda.set_device(0)
    c.init(0)
    return c


def _int(a):
    return int.from_bytes(np.ascontiguousarray(a, dtype="<u4").tobytes(), "little")


def _operand(rng, n, kind):
    if kind == "ones":
        return np.full(n, 0xFFFFFFFF, dtype=np.uint32)
    x = rng.integers(0, 2**32, size=n, dtype=np.uint64).astype(np.uint32)
    if kind == "high":   # every 64-bit digit near 2^64: the largest residues' neighbours
        x |= np.uint32(0xFFFFFF00)
    return x


@pytest.mark.parametrize("k", range(8, 17))
def test_products_around_a_power_of_two(cat, k):
    """One-workgroup transforms of 2^(k-1) digits (k <= 14) and the first
    four-step ones: odd lengths on either side (the last digit half empty),
    la + lb = 2^k + 1 (no coefficient at the top), operands longer than half
    the transform, one-limb operands, tiles that are not full."""
    rng = np.random.default_rng(k)
    n = 1 << k
    pairs = [(n // 2, n // 2), (n // 2 + 1, n // 2), (n // 2 - 1, n // 2 + 1), (n // 2, n // 2 - 1),
             (n - n // 8, n // 8), (n - n // 8 + 1, n // 8), (n - 1, 2), (n, 1), (n // 2 + 3, n // 3)]
    la, lb, a, b = [], [], [], []
    for kind in ("rand", "ones", "high"):
        for x, y in pairs:
            la.append(x)
            lb.append(y)
            a.append(_operand(rng, x, kind))
            b.append(_operand(rng, y, kind))
    a_off = np.concatenate([[0], np.cumsum(la)]).astype(np.uint64)
    b_off = np.concatenate([[0], np.cumsum(lb)]).astype(np.uint64)
    expect = [_int(x) * _int(y) for x, y in zip(a, b)]
    fa, fb = cat.from_numpy(np.concatenate(a)), cat.from_numpy(np.concatenate(b))
    try:
        for fused in (None, 0):   # the short buckets fused, and each in launches of its own
            cat.set_fused_levels(fused)
            print("k", k, "fused", fused, flush=True)
            c, c_off = cat.mul_batched(fa, a_off, fb, b_off)
            got = cat.to_numpy(c)
            for i, e in enumerate(expect):
                assert _int(got[int(c_off[i]):int(c_off[i + 1])]) == e, (k, fused, i, la[i], lb[i])
    finally:
        cat.set_fused_levels(None)


@pytest.mark.parametrize("log_row", [10, 11, 12, 13])
@pytest.mark.parametrize("log_pass", [4, 9, 10])
def test_rows_and_column_passes(cat, log_row, log_pass):
    """Transforms of 2^15 to 2^20 digits under every row and column length that
    the schedule table can ask for."""
    rng = np.random.default_rng(100 * log_row + log_pass)
    base = cat.get_tuning()
    t = {k: (list(v) if isinstance(v, list) else v) for k, v in base.items()}
    for k in range(16, 22):
        t["cls"][k], t["log_row"][k], t["log_pass"][k] = 2, log_row, log_pass
    m = [2**32 - 5, 2**32 + 1, 2**32 - 1]
    try:
        cat.set_tuning(t)
        for k in range(16, 22):
            n = 1 << k
            for x, y, kind in [(n // 2, n // 2, "ones"), (n // 2 + 1, n // 2 - 5, "rand"), (n - 777, 776, "high")]:
                print("rows", log_row, log_pass, k, x, y, kind, flush=True)
                a, b = cat.from_numpy(_operand(rng, x, kind)), cat.from_numpy(_operand(rng, y, kind))
                c, _ = cat.mul_batched(a, [0, x], b, [0, y])
                ra, rb, rc = cat.residues(a), cat.residues(b), cat.residues(c)
                assert [p * q % z for p, q, z in zip(ra, rb, m)] == list(rc), (log_row, log_pass, k, x, y)
    finally:
        cat.set_tuning(base)
