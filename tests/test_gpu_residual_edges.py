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
