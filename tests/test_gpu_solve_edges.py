"""The triangular solves at the edges of their blocking: a given factor L
(unit diagonal, N(0, 1/(16 n)) entries below it) is imported and
X = L^{-T} L^{-1} B is compared with numpy's binary64 solution.

Bound: each substitution with rounded factor and explicit block inverses has
a forward error of at most about 2 n u kappa(L), kappa(L) = || |L^{-1}| |L| ||_inf,
and the first one's error is carried through the second:
4 n u kappa(L) kappa(L^T) relative to max|x|, u the factor's unit roundoff.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
U = {"fp32": 2.0 ** -24, "fp64": 2.0 ** -53}


def check(spd, n, m, prec):
    import torch
    print(f"solve edges n={n} m={m} {prec}", flush=True)
    sys.stdout.flush()
    rng = np.random.Generator(np.random.PCG64(n * 100 + m))
    L = np.tril(rng.standard_normal((n, n)) / (4 * np.sqrt(n)), -1) + np.eye(n)
    B = rng.standard_normal((m, n))
    Li = np.linalg.inv(L)
    ref = (Li.T @ (Li @ B.T)).T
    kap = (np.abs(Li) @ np.abs(L)).sum(axis=1).max() * (np.abs(Li.T) @ np.abs(L.T)).sum(axis=1).max()
    F, info, st = spd.factor_import(torch.from_numpy(L).cuda(), prec=prec)
    assert info == 0 and st == 0
    X = spd.solve(F, torch.from_numpy(B).cuda()).cpu().numpy()
    F.close()
    err = np.abs(X - ref).max(axis=1) / np.abs(ref).max(axis=1)
    assert err.max() <= 4 * n * U[prec] * kap, (err.max(), 4 * n * U[prec] * kap)
    # a wrong or missing block shows as an error of the size of an entry of L
    assert err.max() <= (1e-3 if prec == "fp32" else 1e-11), err.max()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 33, 128, 129, 256, 300, 512, 640, 897, 1024, 1025, 1536, 1700])
def test_block_inverses(spd, n, prec):
    """Orders around the doubling levels of the block inverses (128, 256, 512,
    1024), with whole, ragged and single-block pairs at each level."""
    check(spd, n, 1, prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 128, 129, 1024, 1025, 2048, 2200, 3300])
@pytest.mark.parametrize("m", [2, 3, 16, 17, 32, 35])
def test_many_right_hand_sides(spd, n, m, prec):
    """The VALU (up to 2) and MFMA solves: column tiles and launches (16, 32)
    with ragged ends, one to four big blocks with a whole or short last one."""
    check(spd, n, m, prec)


@pytest.mark.parametrize("n,prec", [(300, "fp32"), (1300, "fp32"), (6000, "fp32"), (300, "fp64"), (1300, "fp64")])
def test_many_columns_round_no_worse_than_one(spd, n, prec):
    """The rounding error of 32 columns solved together against that of the
    same columns one by one.  Both kernels add a block's products in sums of 32
    and these in pairs, so the rms errors agree up to sampling (about 3 % for
    32 columns): at most 1.15 times.  (One sum of 128 per wave gives 1.3 times
    at n = 300, one over all blocks more with every block.)"""
    import torch
    print(f"solve rounding n={n} {prec}", flush=True)
    sys.stdout.flush()
    rng = np.random.Generator(np.random.PCG64(n))
    L = np.tril(rng.standard_normal((n, n)) / (2 * np.sqrt(n)), -1).astype(np.float32).astype(np.float64) + np.eye(n)
    B = rng.standard_normal((32, n)).astype(np.float32).astype(np.float64)
    if prec == "fp32":
        dL = torch.from_numpy(L).cuda()
        ref = torch.cholesky_solve(torch.from_numpy(np.ascontiguousarray(B.T)).cuda(), dL).t().cpu().numpy()
    else:
        ref, M = B.T.astype(np.longdouble), L.astype(np.longdouble)
        for i in range(n):
            ref[i + 1:] -= M[i + 1:, i:i + 1] * ref[i]
        for i in range(n - 1, -1, -1):
            ref[:i] -= M[i:i + 1, :i].T * ref[i]
        ref = ref.T
    F, info, st = spd.factor_import(torch.from_numpy(L).cuda(), prec=prec)
    assert info == 0 and st == 0
    dB = torch.from_numpy(B).cuda()
    many = spd.solve(F, dB).cpu().numpy()
    one = np.concatenate([spd.solve(F, dB[c:c + 1]).cpu().numpy() for c in range(32)])
    F.close()
    e_many, e_one = (float(np.linalg.norm((X - ref).astype(np.float64))) for X in (many, one))
    print(f"  {e_many / e_one:.3f}", flush=True)
    assert e_many <= 1.15 * e_one, (e_many, e_one)
