"""The binary64 residual at the edges of its kernels' tiles, slices and
dispatch (two right-hand sides | more; 16 and 32 columns per pass), with a
leading dimension larger than n and NaN wherever A must not be read (above
the diagonal, beyond n).  Bound as in the parity tests:
|R - R_oracle| <= (n + 1) u (|A| |X| + |B|) elementwise."""
import sys

import numpy as np
import pytest

import spdgen

pytestmark = pytest.mark.gpu
U64 = 2.0 ** -53


@pytest.mark.parametrize("n", [1, 2, 15, 63, 64, 65, 127, 128, 129, 200, 257, 385, 1029])
@pytest.mark.parametrize("m", [1, 2, 3, 8, 16, 17, 32, 33, 49])
def test_residual_edges(spd, orc, n, m):
    _edge(spd, orc, n, m, pad=1 + (n + m) % 4)


@pytest.mark.parametrize("n,m", [(2880, 1), (2944, 2), (2945, 1), (4100, 1)])
def test_residual_tiles_per_workgroup(spd, orc, n, m):
    """Orders on both sides of the rule that gives a workgroup of the single
    pass more than one tile in sequence (n > 2880)."""
    _edge(spd, orc, n, m, pad=0)


def _edge(spd, orc, n, m, pad):
    import torch
    print(f"residual edges n={n} m={m} lda={n + pad}", flush=True)
    sys.stdout.flush()
    rng = np.random.Generator(np.random.PCG64(1000 * n + m))
    A = rng.standard_normal((n, n))
    A = A + A.T
    X, Bt = rng.standard_normal((m, n)), rng.standard_normal((m, n))
    P = np.full((n, n + pad), np.nan)  # row j = column j of the column-major matrix
    for j in range(n):
        P[j, j:n] = A[j:, j]
    dA = torch.from_numpy(P).cuda()[:, :n].t()  # stride (1, n + pad)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    R, eta = spd.residual(dA, dev(X), dev(Bt))
    R = R.cpu().numpy()
    Ro = orc.residual(A, X, Bt)
    bound = (n + 1) * U64 * (np.abs(X) @ np.abs(A) + np.abs(Bt))
    assert np.all(np.abs(R - Ro) <= bound)
    want = np.abs(R).max(axis=1) / (np.abs(A).sum(axis=1).max() * np.abs(X).max(axis=1) + np.abs(Bt).max(axis=1))
    assert np.allclose(eta, want, rtol=1e-12, atol=0)


# rms rounding error in units of u |a||x| sqrt(n) (rms values) on the inputs
# below of the kernels before the single pass took fewer tiles per workgroup
# and the many-column one to registers: one column, three or more
FORMER = {300: (0.612, 0.700), 700: (0.788, 1.086), 1300: (0.901, 1.536), 2500: (1.065, 2.084), 4000: (1.254, 2.156),
          6000: (1.372, 3.385)}


@pytest.mark.parametrize("n", sorted(FORMER))
@pytest.mark.parametrize("m", [1, 3, 8, 32])
def test_residual_rounding(spd, n, m):
    """The rounding error of A X against the exact one in whole numbers, no
    larger than it has been (10 % for the sampling)."""
    import torch
    g = torch.Generator(device="cuda")
    sq = count = 0
    for seed in range(max(1, 6000 // n)):
        g.manual_seed(1000 * n + seed)
        A = torch.randint(-2 ** 24, 2 ** 24, (n, n), device="cuda", generator=g)
        A = torch.tril(A) + torch.tril(A, -1).t()
        X = torch.randint(-2 ** 26, 2 ** 26, (m, n), device="cuda", generator=g)  # sums below 2^63
        R = spd.residual(A.double(), X.double(), torch.zeros(m, n, dtype=torch.float64, device="cuda"))[0]
        for c in range(min(m, 3)):
            exact = -(A * X[c]).sum(1)
            hi = exact.double()
            sq += float((((R[c] - hi) - (exact - hi.long()).double()) ** 2).sum())
            count += n
    err = (sq / count) ** 0.5 / (2.0 ** 50 / 3 * n ** 0.5 * U64)
    print(f"residual rounding n={n} m={m}: {err:.3f}", flush=True)
    assert err <= 1.1 * FORMER[n][0 if m == 1 else 1], err
