"""What the speed of this library is judged on: a list of calls, and ranges from which more of them can be drawn.

A case is one call of a tensor-level entry point of the package (recurrence_matmul, recurrence_trsm,
recurrence_cholesky, recurrence_attention) on random data of the kind that the benchmark and the tests use.  The large
ones are the sizes that bench.py measures; the others are what the same programs call besides: small products in which
a launch is most of the time, sizes that are no multiple of anything, few right-hand sides, one query against a long
list of keys.
"""
from __future__ import annotations

import math

import torch

import paper_2511_09987_amd as lib

DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------ cases
def _matmul(dtype, batch, M, K, N):
    return {"op": "matmul", "dtype": dtype, "batch": batch, "M": M, "K": K, "N": N}


def _trsm(n, nrhs, nb=64):
    return {"op": "trsm", "n": n, "nrhs": nrhs, "nb": nb}


def _cholesky(n, nb=64):
    return {"op": "cholesky", "n": n, "nb": nb}


def _attention(batch, N, M, d):
    return {"op": "attention", "batch": batch, "N": N, "M": M, "d": d}


def listed():
    table = {
        # the smallest product: one grid of 64 x 64 cells, all latency
        "matmul_i8_64": _matmul("i8", 1, 64, 64, 64),
        # an ordinary small product, as in the inner loop of a blocked algorithm
        "matmul_bf16_512": _matmul("bf16", 1, 512, 512, 512),
        # sizes that come from data and not from a tile: no row of A or B starts at a 16-byte boundary
        "matmul_bf16_odd": _matmul("bf16", 1, 3001, 2999, 3003),
        # the large products, one of each element type
        "matmul_bf16_8192": _matmul("bf16", 1, 8192, 8192, 8192),
        "matmul_i8_8192": _matmul("i8", 1, 8192, 8192, 8192),
        # weights that dwarf what streams past them: 32 weight matrices, 16 columns each
        "matmul_bf16_narrow": _matmul("bf16", 32, 8192, 8192, 16),
        # few outputs and a long sum (a weight gradient over many samples)
        "matmul_bf16_tall_k": _matmul("bf16", 1, 512, 262144, 512),
        # forward solve with many right-hand sides, and a small one whose last tile and last slab are ragged
        "trsm_8192": _trsm(8192, 8192),
        "trsm_1000x136": _trsm(1000, 136),
        # factorisation of a large matrix
        "cholesky_8192": _cholesky(8192),
        # attention over whole sequences (batch x heads = 64), and one new query per head against 4000 keys
        "attention_4096": _attention(64, 4096, 4096, 128),
        "attention_one_query": _attention(64, 1, 4000, 128),
    }
    return [dict(case, name=name) for name, case in table.items()]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _round_to(x, step):
    return max(step, (x + step // 2) // step * step)


def draw(rng):
    kind = rng.choice(["product", "product", "product_odd", "product_odd", "narrow", "few_rows", "tall_k", "trsm", "trsm",
                       "cholesky", "cholesky", "attention", "attention", "queries"])
    dtype = rng.choice(["bf16", "bf16", "i8"])
    step = 16 if dtype == "i8" else 8
    if kind == "product":             # rows of A and B start at 16-byte boundaries
        while True:
            M, K, N = _log_int(rng, 16, 8192), _round_to(_log_int(rng, 32, 8192), step), _round_to(_log_int(rng, 16, 8192), step)
            batch = rng.choice([1, 1, 1, 2, 5, 16])
            if 2.0 * batch * M * K * N <= 1.1e12:
                return _matmul(dtype, batch, M, K, N)
    if kind == "product_odd":         # and where they do not
        while True:
            M, K, N = _log_int(rng, 16, 4096), _log_int(rng, 16, 4096) | 1, _log_int(rng, 16, 4096) | rng.choice([0, 1])
            batch = rng.choice([1, 1, 1, 3])
            if 2.0 * batch * M * K * N <= 5.4e10:
                return _matmul(dtype, batch, M, K, N)
    if kind == "narrow":
        return _matmul(dtype, rng.choice([1, 2, 8, 32]), _log_int(rng, 4096, 8192), _round_to(_log_int(rng, 1024, 8192), step),
                       rng.randint(1, 16))
    if kind == "few_rows":
        return _matmul(dtype, rng.choice([1, 2, 8, 32]), rng.randint(1, 32), _round_to(_log_int(rng, 1024, 8192), step),
                       _round_to(_log_int(rng, 1024, 8192), step))
    if kind == "tall_k":
        return _matmul(dtype, 1, _log_int(rng, 16, 1024), _round_to(_log_int(rng, 4096, 131072), 64),
                       _round_to(_log_int(rng, 16, 1024), step))
    if kind == "trsm":
        n, nrhs = _log_int(rng, 64, 8192), _log_int(rng, 8, 8192)
        if rng.random() < 0.75:       # the usual alignment
            n, nrhs = _round_to(n, 8), _round_to(nrhs, 8)
        elif n > 2048:
            n //= 4
        return _trsm(n, nrhs, rng.choice([64, 64, 64, 64, 32, 128]) if n <= 2048 else 64)
    if kind == "cholesky":
        n = _log_int(rng, 64, 8192)
        if rng.random() < 0.75:
            n = _round_to(n, 8)
        elif n > 2048:
            n //= 4
        return _cholesky(n, rng.choice([64, 64, 64, 32]) if n <= 2048 else 64)
    if kind == "attention":
        N = _log_int(rng, 64, 4096)
        M = N if rng.random() < 0.5 else _log_int(rng, 64, 4096)
        return _attention(_log_int(rng, 1, 64), N, M, rng.choice([64, 128]))
    return _attention(_log_int(rng, 1, 64), rng.randint(1, 16), _log_int(rng, 128, 16384), rng.choice([64, 128]))


# ------------------------------------------------------------------------------------------------ inputs
def _normal(shape, sigma, gen, dtype):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    for s in range(0, flat.numel(), 1 << 28):
        part = flat[s:s + (1 << 28)]
        part.normal_(0.0, sigma, generator=gen)
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    op = case["op"]
    if op == "matmul":
        b, M, K, N = case["batch"], case["M"], case["K"], case["N"]
        sa, sb = ((b, M, K), (b, K, N)) if b > 1 else ((M, K), (K, N))
        if case["dtype"] == "i8":
            A = torch.randint(-127, 128, sa, dtype=torch.int8, device=DEV, generator=gen)
            B = torch.randint(-127, 128, sb, dtype=torch.int8, device=DEV, generator=gen)
        else:                         # variance 1/sqrt(K): results of unit variance
            A = _normal(sa, K ** -0.25, gen, torch.bfloat16)
            B = _normal(sb, K ** -0.25, gen, torch.bfloat16)
        return op, A, B
    if op == "trsm":                  # a well-conditioned lower triangle, zero above
        n, nrhs = case["n"], case["nrhs"]
        L = _normal((n, n), 0.5 / math.sqrt(n), gen, torch.bfloat16).tril_(-1)
        L.diagonal().copy_(1.0 + torch.rand(n, device=DEV, generator=gen))
        return op, L, _normal((n, nrhs), 1.0, gen, torch.float32), case["nb"]
    if op == "cholesky":              # symmetric, eigenvalues in about [1.5, 4.5]
        n = case["n"]
        G = _normal((n, n), 0.5 / math.sqrt(n), gen, torch.float32).tril_(-1)
        A = G + G.t()
        A.diagonal().copy_(2.5 + torch.rand(n, device=DEV, generator=gen))
        return op, A, case["nb"]
    b, N, M, d = case["batch"], case["N"], case["M"], case["d"]
    return op, _normal((b, N, d), 1.0, gen, torch.bfloat16), _normal((b, M, d), 1.0, gen, torch.bfloat16), \
        _normal((b, M, d), 1.0, gen, torch.bfloat16)


def run(state):
    op = state[0]
    if op == "matmul":
        return lib.recurrence_matmul(state[1], state[2])
    if op == "trsm":
        return lib.recurrence_trsm(state[1], state[2], state[3])
    if op == "cholesky":
        return lib.recurrence_cholesky(state[1], state[2])
    return lib.recurrence_attention(state[1], state[2], state[3])


# ------------------------------------------------------------------------------------------------ work and tolerance
def work(case):
    op = case["op"]
    if op == "matmul":
        b, M, K, N = case["batch"], case["M"], case["K"], case["N"]
        es = 1 if case["dtype"] == "i8" else 2
        return {"bytes": b * ((M * K + K * N) * es + 4 * M * N), "flops": 2 * b * M * K * N}
    if op == "trsm":                  # lower triangle of L and B in, X and its bfloat16 rounding out
        n, nrhs = case["n"], case["nrhs"]
        return {"bytes": n * (n + 1) + n * nrhs * 10, "flops": n * (n + 1) * nrhs}
    if op == "cholesky":              # lower triangle of A in, L and its bfloat16 rounding (whole squares) out
        n = case["n"]
        return {"bytes": n * (n + 1) // 2 * 4 + n * n * 6, "flops": n ** 3 // 3}
    b, N, M, d = case["batch"], case["N"], case["M"], case["d"]
    return {"bytes": b * ((N + 2 * M) * d * 2 + N * d * 4), "flops": 4 * b * N * M * d}


def tolerance(case):
    """Each bound is four to five times what was measured against 64-bit sums (matmul, attention), or between the two orders
    of summation and the two ways through a diagonal tile that the library itself has (trsm, cholesky)."""
    op = case["op"]
    if op == "matmul":                # products are exact; fp32 sums: 1e-7 .. 6e-7 for K of 512 .. 262144
        return "exact" if case["dtype"] == "i8" else {"rel": 3e-6}
    if op == "trsm":                  # a last-bit difference tips a bfloat16 rounding here and there: 2e-5 in X, 1.7e-4 in its rounding
        return {"rel": 7e-4}
    if op == "cholesky":              # likewise: 8e-7 in L, 1.4e-5 in its rounding at n = 4096, growing with n
        return {"rel": 1e-4}
    return {"rel": 7e-3}              # weights rounded to bfloat16: 1.4e-3 .. 1.8e-3


# ------------------------------------------------------------------------------------------------ 64-bit results
def exact(case, seed):
    """What run() returns, from the definition in 64 bits.  The rounding of X and L to bfloat16 that trsm and cholesky also
    return is compared with the unrounded result; above the diagonal that copy of L is its mirror image."""
    op = case["op"]
    state = prepare(case, seed)
    if op == "matmul":
        A, B = state[1], state[2]
        if A.dim() == 2:
            return torch.matmul(A.double(), B.double())
        return torch.stack([torch.matmul(a.double(), b.double()) for a, b in zip(A, B)])
    if op == "trsm":
        X = torch.linalg.solve_triangular(state[1].double(), state[2].double(), upper=False)
        return X, X
    if op == "cholesky":
        L = torch.linalg.cholesky(state[1].double())
        return L, L + L.tril(-1).t()
    out = []
    for q, k, v in zip(*(t.double() for t in state[1:])):
        out.append(torch.matmul(torch.softmax(torch.matmul(q, k.t()) / math.sqrt(case["d"]), -1), v))
    return torch.stack(out)
