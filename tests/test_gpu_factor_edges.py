"""The factorisation at the edges of its tiles: orders around the 16-column
halves and 32-column strips of a diagonal block, around whole panels and (in
binary64) around the 64- and 128-row tiles of the trailing update, each
against its own backward error bound |H - L L^T| <= 4 (n + 1) u |L||L^T|
elementwise, as in the parity tests; and the breakdown column at the first and
last columns of halves, strips and panels, which has to be the oracle's."""
import numpy as np
import pytest

import spdgen
from test_gpu_parity import _say, dev, host

pytestmark = pytest.mark.gpu
U = {"fp32": 2.0 ** -24, "fp64": 2.0 ** -53}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 48, 65, 97, 127, 128, 129, 161, 256, 385, 640, 1153])
def test_backward_error(spd, n, prec):
    _say(f"factor edges {prec} n={n}")
    A = spdgen.logspaced(n, 1e2, 700 + n)
    F, info, st = spd.factor(dev(A), prec)
    assert info == 0 and st == 0
    L, d, mu = spd.export(F)
    L, d = host(L), host(d)
    F.close()
    H = (((d[:, None] * A) * d[None, :]).astype(np.float32).astype(np.float64)) if prec == "fp32" else A
    assert np.count_nonzero(np.triu(L, 1)) == 0
    E = np.abs(H - L @ L.T)
    assert np.all(E <= 4 * (n + 1) * U[prec] * (np.abs(L) @ np.abs(L.T))), np.max(E)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_breakdown_columns(spd, orc, prec):
    n = 300
    for j0 in (1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65, 80, 96, 97, 112, 113, 127, 128, 129, 144, 145, 256,
               272, 273, 300):
        _say(f"breakdown edges {prec} j0={j0}")
        A = spdgen.indefinite(n, j0, seed=90 + j0)
        F, info, st = spd.factor(dev(A), prec)
        if F is not None:
            F.close()
        assert st == spd.ERR_NOT_SPD and info == j0, (j0, info, st)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("j0", [1, 2, 15, 16, 17, 32, 33, 128, 129, 200])
def test_zero_pivot(spd, prec, j0):
    """A pivot that is exactly zero (its row and column zero as well)."""
    n = 200
    A = np.array(spdgen.logspaced(n, 1e1, 40 + j0))
    A[j0 - 1, :] = A[:, j0 - 1] = 0.0
    _say(f"zero pivot {prec} j0={j0}")
    F, info, st = spd.factor(dev(A), prec)
    F.close()
    assert st == spd.ERR_NOT_SPD and info == j0, (info, st)


@pytest.mark.parametrize("k", [100, -500, 480, 500, 505, 510, 520])
def test_power_of_four_scales_through(spd, k):
    """Roots and quotients of the binary64 diagonal block keep their bits over
    the whole range: A 4^-k has the factor L 2^-k, exactly, for 2 x 2 blocks of
    few-bit numbers (subnormal ones, too, for k = 510 and 520)."""
    n = 192
    rng = np.random.Generator(np.random.PCG64(5))
    A = np.zeros((n, n))
    for i in range(0, n, 2):
        p, q, r = rng.integers(2 ** 17, 2 ** 19), rng.integers(1, 2 ** 16), rng.integers(2 ** 18, 2 ** 19)
        A[i, i], A[i + 1, i], A[i, i + 1], A[i + 1, i + 1] = p, q, q, r
    A *= 2.0 ** -18
    _say(f"factor scaled by 4^-{k}")

    def factor(M):
        F, info, st = spd.factor(dev(M), "fp64")
        L = host(spd.export(F)[0])
        F.close()
        assert info == 0 and st == 0
        return L

    L, S = factor(A), factor(A * 2.0 ** (-2 * k))
    want = L * 2.0 ** -k
    if k < 505:  # beyond, what comes off the second pivot is itself rounded as a subnormal
        assert np.array_equal(S, want), np.argwhere(S != want)[:5]
    i = np.arange(0, n, 2)
    assert np.array_equal(S[i, i], want[i, i]) and np.array_equal(S[i + 1, i], want[i + 1, i])
