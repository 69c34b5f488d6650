"""Timed cases of the public entry points, over the sizes a user's program has.

listed() names the cases, draw() gives more of the same ranges, prepare()
builds on the GPU what a program holds before the call (inputs from the seed,
output buffers, plans), run() is one pass through the package's entry points
and returns its whole output, work() the bytes and operations that no
implementation can do without, exact() the outputs from Python's integers where
that is quick.

Every output is a whole number (limbs of 32 bits in int32 tensors, or ASCII
digits), so there is nothing to round.
"""
import math
import sys

import numpy as np
import torch

import paper_2601_11621_amd as cat

# The largest n that the method was published for (its Table 1).
N_LARGEST = 2_050_572_903


def listed():
    return [
        # one small request: everything is latency and launches
        {"name": "catalan_1e3", "kind": "catalan", "n": 1_000},
        # an ordinary request of a service
        {"name": "catalan_1e5", "kind": "catalan", "n": 100_000},
        # the published table's sizes (10^7 and 10^8), and its largest run
        {"name": "catalan_1e7", "kind": "catalan", "n": 10_000_000},
        {"name": "catalan_1e8", "kind": "catalan", "n": 100_000_000},
        {"name": "catalan_largest", "kind": "catalan", "n": N_LARGEST},
        # eight waiting requests of mixed sizes answered as one batch
        {"name": "serve_8", "kind": "serve", "count": 8, "lo": 1_000, "hi": 10_000_000},
        # a binomial coefficient (a factorial ratio whose exponents are not C(n)'s)
        {"name": "binomial_2e7", "kind": "binomial", "n": 20_000_000, "k": 10_000_000},
        # rebuilding a number from a factorisation that is already there
        {"name": "rebuild_3e7", "kind": "rebuild", "n": 30_000_000},
        # one level of a product tree of uneven nodes, under a kept plan
        {"name": "level_4096", "kind": "level", "count": 4096, "lo_log2": 6.0, "hi_log2": 16.0},
        # a few short products in one call, lengths new to the caller
        {"name": "products_short", "kind": "products", "count": 48, "la": 777, "lb": 301},
        # one long product of ragged lengths
        {"name": "product_long", "kind": "products", "count": 1, "la": 5_000_011, "lb": 3_000_017},
        # decimal text of a number of C(10^8)'s length
        {"name": "decimal_6249999", "kind": "decimal", "limbs": 6_249_999},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["catalan", "catalan", "serve", "binomial", "rebuild", "level", "products", "products", "decimal"])
    if kind == "catalan":
        return {"kind": kind, "n": min(_log_uniform(rng, 1_000, N_LARGEST), N_LARGEST)}
    if kind == "serve":
        lo = _log_uniform(rng, 1_000, 100_000)
        return {"kind": kind, "count": rng.randint(2, 16), "lo": lo, "hi": _log_uniform(rng, 2 * lo, 10_000_000)}
    if kind == "binomial":
        n = _log_uniform(rng, 2_000, 100_000_000)
        return {"kind": kind, "n": n, "k": rng.randint(n // 8, n // 2)}
    if kind == "rebuild":
        return {"kind": kind, "n": _log_uniform(rng, 1_000, 200_000_000)}
    if kind == "level":
        lo = rng.uniform(4.0, 10.0)
        return {"kind": kind, "count": _log_uniform(rng, 16, 4096), "lo_log2": round(lo, 3),
                "hi_log2": round(rng.uniform(lo + 1.0, 16.0), 3)}
    if kind == "products":
        count = _log_uniform(rng, 1, 256)
        most = 8_000_000 // count
        return {"kind": kind, "count": count, "la": _log_uniform(rng, 1, most), "lb": _log_uniform(rng, 1, most)}
    return {"kind": kind, "limbs": _log_uniform(rng, 50, 6_500_000)}


# ---------------------------------------------------------------------------
# Inputs.  C(n), binomials and factorisations have no input but their numbers:
# the seed moves n down by less than 48, among those whose results have equally
# many limbs (so that outputs of two seeds have one shape).


def _log2_binomial(n, k):
    return (math.lgamma(n + 1) - math.lgamma(k + 1) - math.lgamma(n - k + 1)) / math.log(2)


def _shifted(n, seed, bits=lambda n: _log2_binomial(2 * n, n) - math.log2(n + 1)):
    by_limbs = {}
    for m in range(n - 47, n + 1):
        by_limbs.setdefault(int(bits(m) // 32), []).append(m)
    most = max(by_limbs.values(), key=len)
    return most[seed % len(most)]


def _limbs(count, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(-(2**31), 2**31, (count,), dtype=torch.int32, device="cuda", generator=g)


def _lengths(case):
    """The operand lengths of a batch: part of the case, as of a kept plan."""
    if case["kind"] == "level":
        rng = np.random.default_rng(case["count"])
        lens = [np.rint(2 ** rng.uniform(case["lo_log2"], case["hi_log2"], case["count"])).astype(np.int64)
                for _ in range(2)]
    else:
        # ragged: product i is i % 7 and i % 5 limbs shorter, down to one
        i = np.arange(case["count"])
        lens = [np.maximum(case["la"] - i % 7, 1), np.maximum(case["lb"] - i % 5, 1)]
    return [np.concatenate([[0], np.cumsum(x)]).astype(np.uint64) for x in lens]


def _requests(case, seed=0):
    """Sizes of a batch of requests, spread evenly over their logarithm."""
    c, lo, hi = case["count"], case["lo"], case["hi"]
    ns = [int(lo * (hi / lo) ** (i / max(1, c - 1))) for i in range(c)]
    return [_shifted(n, seed) for n in ns]


def _binomial(case, seed):
    k = min(case["k"], (case["n"] - 47) // 2)
    return _shifted(case["n"], seed, lambda n: _log2_binomial(n, k)), k


def prepare(case, seed):
    cat.init(torch.cuda.current_device())
    kind = case["kind"]
    if kind == "catalan":
        n = _shifted(case["n"], seed)
        return {"kind": kind, "n": n, "out": torch.empty(cat.sizes(n)[1], dtype=torch.int32, device="cuda")}
    if kind == "serve":
        return {"kind": kind, "ns": _requests(case, seed)}
    if kind == "binomial":
        n, k = _binomial(case, seed)
        return {"kind": kind, "num": [n], "den": [k, n - k],
                "out": torch.empty(cat.ratio_sizes([n], [k, n - k])[1], dtype=torch.int32, device="cuda")}
    if kind == "rebuild":
        exps, off, primes = cat.factor(_shifted(case["n"], seed))
        return {"kind": kind, "exps": exps, "off": off, "primes": primes.clone(),
                "out": torch.empty(cat.product_sizes(exps, off)[0], dtype=torch.int32, device="cuda")}
    if kind == "decimal":
        x = _limbs(case["limbs"], seed)
        x[-1] = (1 << 30) + seed % (1 << 20)   # numbers of one length in digits too
        return {"kind": kind, "x": x}
    a_off, b_off = _lengths(case)
    state = {"kind": kind, "a": _limbs(int(a_off[-1]), 2 * seed), "b": _limbs(int(b_off[-1]), 2 * seed + 1),
             "a_off": a_off, "b_off": b_off}
    if kind == "level":
        state["plan"] = cat.MulPlan(a_off, b_off)
        state["c"] = torch.empty(int(a_off[-1] + b_off[-1]), dtype=torch.int32, device="cuda")
    return state


def run(state):
    kind = state["kind"]
    if kind == "catalan":
        return cat.exact(state["n"], out=state["out"])
    if kind == "serve":
        return cat.exact_batch(state["ns"])
    if kind == "binomial":
        return cat.ratio_exact(state["num"], state["den"], out=state["out"])
    if kind == "rebuild":
        return cat.product(state["exps"], state["off"], state["primes"], out=state["out"])
    if kind == "decimal":
        return cat.to_decimal_device(state["x"])
    if kind == "level":
        return state["plan"](state["a"], state["b"], state["c"])
    return cat.mul_batched(state["a"], state["a_off"], state["b"], state["b_off"])[0]


# ---------------------------------------------------------------------------
# Work.  Operations are those of textbook FFT multiplication: the operands cut
# into 16-bit pieces, three real transforms of 2.5 M log2 M operations each
# over the M pieces of the product (or the schoolbook's 2 la lb where that is
# less); a product tree has one such level for every doubling of its nodes.


def _mul_ops(la, lb):
    m = 2.0 * (la + lb)
    return min(2.0 * la * lb, 7.5 * m * math.log2(m))


def _tree_ops(limbs):
    """Every level of the balanced tree over `limbs` one-limb leaves."""
    ops, node = 0.0, 1.0
    while node < limbs:
        ops += limbs / (2 * node) * _mul_ops(node, node)
        node *= 2
    return ops


def _result_limbs(case):
    """Limbs of C(n) (2n bits), or of the binomial (its entropy)."""
    n = case["n"]
    if case["kind"] == "binomial":
        q = case["k"] / n
        return n * -(q * math.log2(q) + (1 - q) * math.log2(1 - q)) / 32
    return 2 * n / 32


def work(case):
    kind = case["kind"]
    if kind in ("catalan", "binomial", "rebuild"):
        limbs = _result_limbs(case)
        primes = 2 * case["n"] / math.log(2 * case["n"])
        read = 4 * primes if kind == "rebuild" else 0
        return {"bytes": 4 * limbs + read, "flops": _tree_ops(limbs)}
    if kind == "serve":
        limbs = [n / 16 for n in _requests(case)]
        return {"bytes": 4 * sum(limbs), "flops": sum(_tree_ops(x) for x in limbs)}
    if kind == "decimal":
        # one byte a digit; a tree of products over the number's halves
        return {"bytes": 4 * case["limbs"] + 9.64 * case["limbs"], "flops": _tree_ops(case["limbs"])}
    a_off, b_off = _lengths(case)
    la, lb = np.diff(a_off.astype(np.int64)), np.diff(b_off.astype(np.int64))
    return {"bytes": 8.0 * float(la.sum() + lb.sum()),
            "flops": sum(_mul_ops(int(x), int(y)) for x, y in zip(la, lb))}


# ---------------------------------------------------------------------------
# The same outputs from Python's integers, where that takes seconds.


def _to_int(x):
    return int.from_bytes(x.cpu().numpy().tobytes(), "little")


def _to_limbs(v, count=None):
    count = count or max(1, -(-v.bit_length() // 32))
    return torch.from_numpy(np.frombuffer(v.to_bytes(4 * count, "little"), dtype=np.int32).copy())


def _catalan(n):
    return math.comb(2 * n, n) // (n + 1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("catalan", "rebuild") and case["n"] <= 200_000:
        return _to_limbs(_catalan(_shifted(case["n"], seed)))
    if kind == "serve" and case["hi"] <= 100_000:
        return [_to_limbs(_catalan(n)) for n in _requests(case, seed)]
    if kind == "binomial" and case["n"] <= 200_000:
        return _to_limbs(math.comb(*_binomial(case, seed)))
    if kind == "decimal" and case["limbs"] <= 10_000:
        sys.set_int_max_str_digits(0)
        text = str(_to_int(prepare(case, seed)["x"]))
        return torch.from_numpy(np.frombuffer(text.encode(), dtype=np.uint8).copy())
    if kind in ("level", "products"):
        a_off, b_off = _lengths(case)
        la, lb = np.diff(a_off.astype(np.int64)), np.diff(b_off.astype(np.int64))
        if float(np.sum(np.maximum(la, lb) * np.minimum(la, lb) ** 0.585)) > 5e8:
            return None
        s = prepare(case, seed)
        a, b = s["a"].cpu().numpy(), s["b"].cpu().numpy()
        out = []
        for i in range(len(la)):
            x = int.from_bytes(a[int(a_off[i]):int(a_off[i + 1])].tobytes(), "little")
            y = int.from_bytes(b[int(b_off[i]):int(b_off[i + 1])].tobytes(), "little")
            out.append(_to_limbs(x * y, int(la[i] + lb[i])))
        return torch.cat(out)
    return None
