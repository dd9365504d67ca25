"""What a program that evaluates encrypted queries has this library do, as
measurable cases: predicate masks, selections, aggregations, comparisons and
joins over batch-encoded columns, through the package's Context.

Sizes.  A column is a number of ciphertexts of 32,768 rows (N = 2^15, the
paper's parameters); the paper's tables have one ciphertext per column, the
benchmark's column has 2^20 rows = 32 ciphertexts, its batched predicates
1 to 32 ciphertexts each.  alpha (data primes per key-switching digit) is 3
by default, 2 and 1 are the other decompositions a context can be made with
(17 data primes and one digit per prime is SEAL's arrangement).  Rings of
2^12 are the size of the allocation-free call's eight ciphertexts.

Values.  An RLWE ciphertext and a switching key are uniform residues to
anyone without the secret key, and the library never holds that key, so
uniform residues are what it meets in earnest; the plaintext values behind
them do not exist on the device.

Every output is an array of whole numbers (residues in [0, q_i)), which an
evaluation determines exactly.
"""
from __future__ import annotations

import math

import torch

from paper_2602_24271_amd import Context
from paper_2602_24271_amd.params import paper_params

DATA_PRIMES = {1: 17, 2: 16, 3: 15}   # the paper's 18 primes, alpha of them special


def listed():
    return [
        # WHERE a = b over the benchmark's column: 2^20 rows, both sides encrypted
        {"name": "eq_column", "op": "eq", "log2_n": 15, "alpha": 3, "n": 32, "broadcast": False},
        # the same over one ciphertext, the paper's 32K-row table: the latency
        # of one predicate
        {"name": "eq_one", "op": "eq", "log2_n": 15, "alpha": 3, "n": 1, "broadcast": False},
        # WHERE a = constant over 150K rows (a last ciphertext partly filled
        # is still a ciphertext), digits of two primes
        {"name": "eq_constant", "op": "eq", "log2_n": 15, "alpha": 2, "n": 5, "broadcast": True},
        # one digit per data prime (SEAL's arrangement), an odd column
        {"name": "eq_one_prime_digits", "op": "eq", "log2_n": 15, "alpha": 1, "n": 11,
         "broadcast": False},
        # a small ring: the eight ciphertexts at 2^12 that the allocation-free
        # call is sized for
        {"name": "eq_small_ring", "op": "eq", "log2_n": 12, "alpha": 1, "n": 8,
         "broadcast": False},
        # predicates of several queries answered together: uneven instances,
        # each against its own constant, in waves
        {"name": "eq_batched", "op": "eq_batched", "log2_n": 15, "alpha": 3,
         "sizes": "1,3,17,2,9,1,7"},
        # WHERE a IN (4 values)
        {"name": "in_set", "op": "in", "log2_n": 15, "alpha": 3, "n": 2, "k": 4},
        # SELECT column WHERE mask on one ciphertext: the smallest product
        {"name": "select_one", "op": "select", "log2_n": 15, "alpha": 3, "n": 1},
        # COUNT or SUM of the benchmark's column: 15 rotations
        {"name": "sum_column", "op": "sum_slots", "log2_n": 15, "alpha": 3, "n": 32},
        # SELECT SUM(column) WHERE mask on a small table
        {"name": "sum_where", "op": "sum_where", "log2_n": 15, "alpha": 3, "n": 3},
        # WHERE a < constant: the comparison polynomial (526 products)
        {"name": "less_than", "op": "less_than", "log2_n": 15, "alpha": 3, "n": 2},
        # equi-join with aggregation against two reference rows
        {"name": "join", "op": "join", "log2_n": 15, "alpha": 3, "n": 2, "rows": "5,20011"},
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    op = rng.choice(["eq", "eq", "eq", "eq_small", "eq_batched", "in", "select", "sum_slots",
                     "sum_where", "less_than", "join"])
    alpha = rng.choice([3, 3, 3, 2, 1])
    if op == "eq":
        # costs grow as alpha falls: the column's 32 ciphertexts at alpha = 3
        # bound the others
        return {"op": "eq", "log2_n": 15, "alpha": alpha,
                "n": _log_int(rng, 1, {3: 32, 2: 26, 1: 19}[alpha]),
                "broadcast": rng.random() < 0.5}
    if op == "eq_small":
        return {"op": "eq", "log2_n": rng.choice([10, 11, 12, 13, 14]), "alpha": alpha,
                "n": _log_int(rng, 1, 16), "broadcast": rng.random() < 0.5}
    if op == "eq_batched":
        sizes, left = [], rng.randint(8, 32)
        while left > 0:
            m = min(left, _log_int(rng, 1, 17))
            sizes.append(m)
            left -= m
        return {"op": "eq_batched", "log2_n": 15, "alpha": 3,
                "sizes": ",".join(str(m) for m in sizes)}
    if op == "in":
        k = rng.randint(2, 6)
        return {"op": "in", "log2_n": 15, "alpha": alpha, "n": _log_int(rng, 1, 18 // k), "k": k}
    if op == "less_than":
        return {"op": "less_than", "log2_n": 15, "alpha": 3, "n": rng.randint(1, 2)}
    if op == "join":
        n_rows = rng.randint(1, 3)
        rows = sorted(rng.sample(range(1 << 15), n_rows))
        return {"op": "join", "log2_n": 15, "alpha": 3, "n": _log_int(rng, 1, 6 // n_rows),
                "rows": ",".join(str(r) for r in rows)}
    # select, sum_slots, sum_where
    return {"op": op, "log2_n": 15, "alpha": alpha, "n": _log_int(rng, 1, 32)}


def _sizes(case):
    return [int(s) for s in case["sizes"].split(",")]


def _rows(case):
    return [int(s) for s in case["rows"].split(",")]


class _Residues:
    """Seeded uniform residues on the device, one limb modulus at a time."""

    def __init__(self, seed, n, device):
        self.gen = torch.Generator(device=device)
        self.gen.manual_seed(seed)
        self.n = n
        self.device = device

    def __call__(self, lead, moduli):
        out = torch.empty((*lead, len(moduli), self.n), dtype=torch.int64, device=self.device)
        for i, m in enumerate(moduli):
            out[..., i, :] = torch.randint(0, int(m), (*lead, self.n), generator=self.gen,
                                           dtype=torch.int64, device=self.device)
        return out


def prepare(case, seed):
    """The context with its keys, and the encrypted operands."""
    p = paper_params(case["log2_n"], alpha=case["alpha"])
    ctx = Context(p["log2_n"], p["t"], p["q"], p["P"], 0)
    rand = _Residues(seed, ctx.n, ctx.device)
    ctx.set_relin_key(rand((ctx.dnum, 2), ctx.moduli_pq))
    state = {"op": case["op"], "ctx": ctx}

    def cts(n):
        return rand((n, 2), ctx.q)

    op = case["op"]
    if op in ("sum_slots", "sum_where", "join"):
        for g in ctx.galois_elements():
            ctx.set_galois_key(g, rand((ctx.dnum, 2), ctx.moduli_pq))
    if op == "eq":
        state["x"] = cts(case["n"])
        state["y"] = cts(1 if case["broadcast"] else case["n"])
    elif op == "eq_batched":
        state["items"] = [(cts(m), cts(1)) for m in _sizes(case)]
    elif op == "in":
        state["x"] = cts(case["n"])
        state["members"] = cts(case["k"])
    elif op in ("select", "sum_where"):
        state["column"] = cts(case["n"])
        state["mask"] = cts(case["n"])
    elif op == "sum_slots":
        state["x"] = cts(case["n"])
    elif op == "less_than":
        state["x"] = cts(case["n"])
        state["y"] = cts(1)
    elif op == "join":
        state["key"] = cts(case["n"])
        state["ref_key"] = cts(1)
        state["ref_attr"] = cts(1)
        state["rows"] = _rows(case)
    return state


def run(state):
    ctx, op = state["ctx"], state["op"]
    if op == "eq":
        return ctx.eq_mask(state["x"], state["y"])
    if op == "eq_batched":
        return ctx.eq_mask_batched(state["items"])
    if op == "in":
        return ctx.in_mask(state["x"], state["members"])
    if op == "select":
        return ctx.select(state["column"], state["mask"])
    if op == "sum_slots":
        return ctx.sum_slots(state["x"])
    if op == "sum_where":
        return ctx.sum_slots(ctx.select(state["column"], state["mask"]))
    if op == "less_than":
        return ctx.compare(state["x"], state["y"], "lt")
    if op == "join":
        return ctx.join_sum(state["key"], state["ref_key"], state["ref_attr"], state["rows"])
    raise ValueError(op)


def work(case):
    """Bytes: operands, keys used and results, once each.  Operations: the
    textbook evaluation's residue arithmetic, a butterfly or a multiply-add
    of residues counted as 8 (a 49-bit product is exact in 6, an add and a
    subtract follow it)."""
    a, log2_n, op = case["alpha"], case["log2_n"], case["op"]
    n, L = 1 << log2_n, DATA_PRIMES[case["alpha"]]
    W, K, dnum = 2 * L + 1, L + a, L // a
    ct = 2 * L * n * 8
    key = dnum * 2 * K * n * 8
    limb = 8 * (n // 2) * log2_n            # one limb's transform
    digits = dnum * K * limb + 8 * n * (dnum * K * (a - 1) + 2 * dnum * K)
    switch = digits + 2 * K * limb + 8 * n * 2 * L * (a + 1)
    lift = 8 * n * 2 * L * (L + 1)          # both polynomials of an operand
    scale = 8 * n * 3 * 2 * L * (L + 1)     # three components, to B and back
    square = lift + 2 * W * limb + 8 * n * 3 * W + 3 * W * limb + scale + switch
    product = square + lift + 2 * W * limb + 8 * n * W
    plain = 4 * L * limb + 8 * n * 2 * L
    k_eq, rotations = 16, 15
    if op == "eq":
        y = 1 if case["broadcast"] else case["n"]
        return {"bytes": (2 * case["n"] + y) * ct + key, "flops": case["n"] * k_eq * square}
    if op == "eq_batched":
        total = sum(_sizes(case))
        return {"bytes": (2 * total + len(_sizes(case))) * ct + key,
                "flops": total * k_eq * square}
    if op == "in":
        return {"bytes": (2 * case["n"] + case["k"]) * ct + key,
                "flops": case["n"] * case["k"] * k_eq * square}
    if op == "select":
        return {"bytes": 3 * case["n"] * ct + key, "flops": case["n"] * product}
    if op == "sum_slots":
        return {"bytes": 2 * case["n"] * ct + rotations * key,
                "flops": case["n"] * rotations * switch}
    if op == "sum_where":
        return {"bytes": 3 * case["n"] * ct + (rotations + 1) * key,
                "flops": case["n"] * (product + rotations * switch)}
    if op == "less_than":
        # 16 squarings, 247 babies and 120 giants (powers of two are squarings),
        # 127 summed tensors with one scaling and one key switch, one product
        parts = 127 * (2 * lift + 4 * W * limb + 8 * n * 4 * W)
        return {"bytes": (2 * case["n"] + 1) * ct + key,
                "flops": case["n"] * (16 * square + 368 * product + parts + 3 * W * limb + scale +
                                      switch + 2 * n * 2 * L * 2 * 256 * 128)}
    if op == "join":
        rows = len(_rows(case))
        spread = 2 * (plain + rotations * switch)
        return {"bytes": (2 * case["n"] + 2) * ct + (rotations + 1) * key,
                "flops": rows * (spread + case["n"] * (k_eq * square + product))}
    raise ValueError(op)
