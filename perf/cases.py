"""Performance cases: solves a user of this library has it do, through the
Python binding's public calls, with inputs made on the GPU from a seed.

Matrices.  "log" is the single-system recipe of `spdgen` (A = Q diag(lambda)
Q^T, eigenvalues log-spaced from 1 to cond) with a Q that is quick to form at
any order: Q = C P S C with C the orthonormal cosine transform, P a seeded
permutation and S seeded signs, so A is dense and has exactly that spectrum.
"cov" is the covariance matrix of the paper's Section 4 (decay d), whose
right-hand sides alone depend on the seed.  Batches have the batched
benchmark's shapes (n ~ U{32..512}, cond ~ 10^U(1, 6), 1..8 right-hand sides
per system); their values depend on the seed.
"""
import math

import numpy as np
import torch

import paper_1405_4644_amd as spd
import spdgen


def listed():
    return [
        # the smallest call: one small system solved on its own, where launches
        # and host round trips are the cost
        {"name": "posv_fp32_n300", "kind": "posv", "prec": "fp32", "matrix": "log", "n": 300, "m": 1, "cond": 1e3},
        # an ordinary system, ragged against every tile, a few right-hand sides
        {"name": "posv_fp32_n1300_m3", "kind": "posv", "prec": "fp32", "matrix": "log", "n": 1300, "m": 3, "cond": 1e4},
        # a mid-size well-conditioned system on a bfloat16 factor
        {"name": "posv_bf16_n3000", "kind": "posv", "prec": "bf16", "matrix": "log", "n": 3000, "m": 1, "cond": 3e1},
        # the headline: the large system with a binary32 factor
        {"name": "posv_fp32_n16384", "kind": "posv", "prec": "fp32", "matrix": "log", "n": 16384, "m": 1, "cond": 1e4},
        # the same order, well conditioned, on a binary16 factor
        {"name": "posv_fp16_n16384", "kind": "posv", "prec": "fp16", "matrix": "log", "n": 16384, "m": 1, "cond": 1e2},
        # the plain binary64 factorisation that the mixed method is held against
        {"name": "posv_fp64_n16384", "kind": "posv", "prec": "fp64", "matrix": "log", "n": 16384, "m": 1, "cond": 1e4},
        # the paper's own workload: covariance matrix, 32 right-hand sides
        {"name": "posv_fp32_cov10000_m32", "kind": "posv", "prec": "fp32", "matrix": "cov", "n": 10000, "m": 32,
         "d": 1},
        # new right-hand sides against a factor kept from before (time stepping, sampling)
        {"name": "resolve_fp32_n6000_m5", "kind": "resolve", "prec": "fp32", "matrix": "log", "n": 6000, "m": 5,
         "cond": 1e3},
        # thousands of small independent systems, binary32 factor
        {"name": "batched_fp32_4096", "kind": "batched", "prec": "fp32", "batch": 4096},
        # the same with the learned picker choosing each system's precision (mostly binary64)
        {"name": "batched_auto_4096", "kind": "batched", "prec": "auto", "batch": 4096},
        # Algorithm 2: conjugate gradients on the dense binary32 operator, one right-hand side
        {"name": "cg_dense_cov10000", "kind": "cg", "matrix": "cov", "n": 10000, "m": 1, "d": 1, "band": -1},
        # Algorithm 2 on the banded operator with the paper's 32 right-hand sides
        {"name": "cg_band16_cov12000_m32", "kind": "cg", "matrix": "cov", "n": 12000, "m": 32, "d": 1, "band": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["posv"] * 5 + ["resolve"] + ["batched"] * 2 + ["cg"] * 2)
    if kind == "posv":
        prec = rng.choice(["fp32", "fp32", "fp32", "fp64", "fp16", "bf16"])
        n = _log_int(rng, 200, 16384)
        m = rng.choice([1, 1, 1, 2, rng.randint(3, 8), rng.randint(9, 32)])
        if rng.random() < 0.25:
            return {"kind": kind, "prec": prec, "matrix": "cov", "n": n, "m": m, "d": rng.choice([1, 2, 4])}
        top = {"fp32": 6.0, "fp64": 6.0, "fp16": 2.2, "bf16": 1.7}[prec]
        return {"kind": kind, "prec": prec, "matrix": "log", "n": n, "m": m, "cond": 10.0 ** rng.uniform(1.0, top)}
    if kind == "resolve":
        return {"kind": kind, "prec": rng.choice(["fp32", "fp32", "fp64"]), "matrix": "log",
                "n": _log_int(rng, 500, 10000), "m": _log_int(rng, 1, 64), "cond": 10.0 ** rng.uniform(1.0, 4.0)}
    if kind == "batched":
        return {"kind": kind, "prec": rng.choice(["fp32", "fp64", "auto", "fp16", "bf16"]),
                "batch": _log_int(rng, 64, 4096)}
    band = rng.choice([-1, rng.randint(4, 32)])
    m = rng.choice([1, 1, rng.randint(2, 8), rng.randint(9, 32)])
    n = _log_int(rng, 1500, 10000 if m == 1 or band >= 0 else 6000)
    # a narrow band converges only where the entries decay fast enough; a slow decay takes many phases
    return {"kind": kind, "matrix": "cov", "n": n, "m": m, "d": rng.choice([1, 2, 4]) if band < 0 or band >= 16 else 4,
            "band": band}


# ---- inputs ---------------------------------------------------------------
def _cosines(n):
    """The orthonormal cosine transform (DCT-II) of order n."""
    j = torch.arange(n, device="cuda")
    C = ((2 * j[None, :] + 1) * j[:, None]).remainder_(4 * n).double().mul_(math.pi / (2 * n)).cos_()
    C.mul_(math.sqrt(2.0 / n))
    C[0].mul_(math.sqrt(0.5))
    return C


def _log_matrices(n, conds, gen):
    """len(conds) matrices of order n with eigenvalues log-spaced from 1 to cond."""
    k = len(conds)
    C = _cosines(n)
    perm = torch.rand(k, n, device="cuda", generator=gen).argsort(dim=1)
    sign = torch.randint(0, 2, (k, n), device="cuda", generator=gen).double().mul_(2).sub_(1)
    Q = C.t()[perm].transpose(1, 2).mul_(sign[:, None, :])  # columns permuted, signs flipped
    Q = torch.matmul(Q.reshape(k * n, n), C).reshape(k, n, n)
    del C
    t = torch.arange(n, dtype=torch.float64, device="cuda") / max(n - 1, 1)
    lam = torch.tensor(conds, dtype=torch.float64, device="cuda")[:, None] ** t[None, :]
    A = torch.bmm(Q * lam[:, None, :], Q.transpose(1, 2).contiguous())
    del Q
    return A.add(A.transpose(1, 2)).mul_(0.5)


def _dense(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, m = case["n"], case["m"]
    if case["matrix"] == "cov":
        A = spdgen.covariance(n, case["d"], backend="torch", device="cuda")
    else:
        A = _log_matrices(n, [case["cond"]], gen)[0]
    X = torch.randn(m, n, dtype=torch.float64, device="cuda", generator=gen)
    return A, X @ A


def _packed(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ns, conds, ms = (np.array(v) for v in zip(*spdgen.batch_shapes(case["batch"])))
    a_off = np.concatenate([[0], np.cumsum(ns * ns)])
    b_off = np.concatenate([[0], np.cumsum(ns * ms)])
    A = torch.empty(int(a_off[-1]), dtype=torch.float64, device="cuda")
    B = torch.empty(int(b_off[-1]), dtype=torch.float64, device="cuda")
    for n in np.unique(ns):
        idx, n = np.nonzero(ns == n)[0], int(n)
        As = _log_matrices(n, [float(c) for c in conds[idx]], gen)
        Bs = torch.matmul(torch.randn(len(idx), 8, n, dtype=torch.float64, device="cuda", generator=gen), As)
        for i, s in enumerate(idx):
            A[a_off[s]:a_off[s + 1]] = As[i].reshape(-1)
            B[b_off[s]:b_off[s + 1]] = Bs[i, :ms[s]].reshape(-1)
    return ns, ms, a_off[:-1], b_off[:-1], A, B


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batched":
        ns, ms, a_off, b_off, A, B = _packed(case, seed)
        dev = [torch.from_numpy(v).to(t).cuda() for v, t in
               ((ns, torch.int32), (ms, torch.int32), (a_off, torch.int64), (b_off, torch.int64))]
        if case["prec"] == "auto":
            spd.picker_load()
        return {"kind": kind, "prec": spd.PREC[case["prec"]],
                "batch": spd.Batch(dev[0], dev[1], dev[2], A, dev[3], B, prec=case["prec"])}
    A, B = _dense(case, seed)
    if kind == "cg":
        return {"kind": kind, "A": A, "B": B, "band": case["band"], "H": spd.CG()}
    if kind == "resolve":
        return {"kind": kind, "A": A, "B": B, "F": spd.factor(A, prec=case["prec"])[0]}
    return {"kind": kind, "A": A, "B": B, "prec": case["prec"], "F": spd.Factor()}


def run(state):
    """One pass: a whole solve, to binary64 accuracy."""
    kind = state["kind"]
    if kind == "posv":
        return spd.posv(state["A"], state["B"], prec=state["prec"], F=state["F"])[0]
    if kind == "resolve":
        X = spd.solve(state["F"], state["B"])
        spd.refine(state["F"], state["A"], state["B"], X)
        return X
    if kind == "batched":
        bt = state["batch"]
        bt.prec.fill_(state["prec"])
        spd.solve_batched(bt)
        return {"X": bt.X, "prec": bt.prec}
    spd.cg_prepare(state["A"], half_band=state["band"], H=state["H"])
    return spd.cg_refine(state["H"], state["A"], state["B"])[0]


def exact(case, seed):
    """The solutions in plain torch binary64: Cholesky, and one step of refinement."""
    def solve(A, B):  # A (..., n, n), B (..., m, n)
        L = torch.linalg.cholesky(A)
        X = torch.cholesky_solve(B.transpose(-1, -2).contiguous(), L)
        X = X + torch.cholesky_solve(B.transpose(-1, -2) - A @ X, L)
        return X.transpose(-1, -2).contiguous()

    if case["kind"] != "batched":
        return solve(*_dense(case, seed))
    ns, ms, a_off, b_off, A, B = _packed(case, seed)
    X = torch.empty_like(B)
    for n in np.unique(ns):
        idx, n = np.nonzero(ns == n)[0], int(n)
        As = torch.stack([A[a_off[s]:a_off[s] + n * n].reshape(n, n) for s in idx])
        Bs = torch.zeros(len(idx), 8, n, dtype=torch.float64, device="cuda")
        for i, s in enumerate(idx):
            Bs[i, :ms[s]] = B[b_off[s]:b_off[s] + n * ms[s]].reshape(-1, n)
        Xs = solve(As, Bs)
        for i, s in enumerate(idx):
            X[b_off[s]:b_off[s] + n * ms[s]] = Xs[i, :ms[s]].reshape(-1)
    return {"X": X, "prec": None}


def work(case):
    """A's lower triangle, B and X once each; the binary64 algorithm's flops
    (a kept factor: the two substitutions; CG: one product and one residual)."""
    if case["kind"] == "batched":
        # expectations over n ~ U{32..512}, m ~ U{1..8}
        n = np.arange(32, 513, dtype=np.float64)
        k, m = case["batch"], 4.5
        return {"bytes": k * float((4 * n * (n + 1) + 16 * n * m).mean()),
                "flops": k * float((n ** 3 / 3 + n ** 2 / 2 + n / 6 + 2 * n ** 2 * m).mean())}
    n, m = float(case["n"]), case["m"]
    byt = 4 * n * (n + 1) + 16 * n * m
    if case["kind"] == "posv":
        return {"bytes": byt, "flops": n ** 3 / 3 + n ** 2 / 2 + n / 6 + 2 * n ** 2 * m}
    if case["kind"] == "resolve":
        elem = 8 if case["prec"] == "fp64" else 4  # the kept factor is read as well
        return {"bytes": byt + elem * n * (n + 1) / 2, "flops": 2 * n ** 2 * m}
    width = n if case["band"] < 0 else 2 * case["band"] + 1
    return {"bytes": byt, "flops": 2 * n ** 2 * m + 2 * width * n * m}
