"""Batched systems at the edges of the kernels' tiles: orders around the last
panel that fits the waves' slots (417 is the first with tiles left over), one
to eight right-hand sides, every precision; and the breakdown column at and
inside both 16-column halves of a diagonal block, which has to be the
oracle's.  Bars as in the batched parity tests."""
import numpy as np
import pytest

import spdgen
from test_gpu_batched import _check_system, _run, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,cond", [("fp32", 1e4), ("fp64", 1e5), ("fp16", 1e1), ("bf16", 1e1)])
def test_tiles_past_the_slots(spd, orc, prec, cond):
    shapes = [(n, cond, m) for n, m in ((15, 3), (17, 8), (48, 1), (415, 2), (416, 8), (417, 1), (447, 5), (448, 3),
                                        (449, 7), (480, 4), (481, 6), (512, 8))]
    _say("batched edges", prec)
    pb = spdgen.packed_batch(shapes, config=3, first_index=3000)
    bt, X, reps, used = _run(spd, pb, prec)
    for s in range(len(shapes)):
        _check_system(orc, pb, s, X, reps[s], prec, prec in ("fp32", "fp64"))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_breakdown_column_in_the_block(spd, orc, prec):
    cols = [1, 2, 15, 16, 17, 18, 31, 32, 33, 48, 49, 64, 80, 81, 96]
    n = 96
    As = [spdgen.indefinite(n, j0, seed=50 + j0) for j0 in cols]
    k = len(cols)
    off = np.arange(k, dtype=np.int64)
    pb = spdgen.PackedBatch(np.full(k, n, np.int32), np.ones(k, np.int32), np.ones(k), off * n * n, off * n,
                            np.concatenate([a.reshape(-1, order="F") for a in As]), np.ones(k * n), np.ones(k * n))
    _say("batched breakdown", prec)
    bt, X, reps, used = _run(spd, pb, prec, spd.default_opts(fallback=0))
    for s, j0 in enumerate(cols):
        assert reps[s]["status"] == spd.ERR_NOT_SPD, (j0, reps[s])
        assert int(reps[s]["info"]) == j0, (j0, reps[s])


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_half_requests_by_themselves_and_falling_back(spd, prec):
    """Half requests have a path of their own in the launch that also holds the
    binary32 ones: the same systems beside binary32 requests give the same
    bits, and what falls back ends as a binary32 request does."""
    shapes = [(n, cond, m) for n, cond, m in ((33, 1e1, 1), (64, 1e6, 3), (130, 1e1, 8), (257, 1e6, 2), (300, 1e1, 4))]
    _say("batched half beside binary32", prec)
    pb = spdgen.packed_batch(shapes, config=3, first_index=6000)
    _, X1, r1, p1 = _run(spd, pb, prec)
    _, X2, r2, p2 = _run(spd, pb, [prec, "fp32", prec, "fp32", prec])
    _, X3, r3, p3 = _run(spd, pb, "fp32")
    assert np.all(r1["status"] == 0) and list(r1["fallbacks"]) == [0, 1, 0, 1, 0], r1
    assert list(p1) == list(p2) and np.array_equal(X1, X2) and np.array_equal(r1["eta"], r2["eta"])
    for s in (1, 3):
        lo, hi = pb.b_off[s], pb.b_off[s] + shapes[s][0] * shapes[s][2]
        assert p1[s] == p3[s] == spd.PREC["fp32"] and np.array_equal(X1[lo:hi], X3[lo:hi])


# geometric mean over 384 systems of the first solve's error in units of u,
# on the inputs below, of the kernels with a left-looking diagonal block
FORMER = {("fp32", 64): 3.827, ("fp32", 128): 4.936, ("fp64", 64): 3.895, ("fp64", 128): 5.158}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("top", [64, 128])
def test_first_solve_rounding(spd, prec, top):
    """The error of one solve without corrections, a few panels deep, no
    larger than it has been (5 %: sampling, 0.7 % rms)."""
    rng = np.random.Generator(np.random.PCG64(top))
    pb = spdgen.packed_batch_grouped([(int(n), 10.0, 2) for n in rng.integers(top // 2, top + 1, 384)], seed=top)
    pb.A, pb.B = pb.A.cpu().numpy(), pb.B.cpu().numpy()
    _, X, reps, _ = _run(spd, pb, prec, spd.default_opts(max_iter=0, fallback=0))
    err = []
    for s in range(384):
        n, a, b = int(pb.n[s]), int(pb.a_off[s]), int(pb.b_off[s])
        A, B = pb.A[a:a + n * n].reshape(n, n), pb.B[b:b + 2 * n].reshape(2, n).T
        x = np.linalg.solve(A, B)
        x = x + np.linalg.solve(A, (B - A.astype(np.longdouble) @ x).astype(np.float64))
        err.append(np.linalg.norm(X[b:b + 2 * n].reshape(2, n).T - x) / np.linalg.norm(x))
    err = float(np.exp(np.mean(np.log(err)))) / (2.0 ** -24 if prec == "fp32" else 2.0 ** -53)
    _say(f"batched rounding {prec} n<={top}: {err:.3f}")
    assert err <= 1.05 * FORMER[prec, top], err


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_half_requests_through_both_fallbacks(spd, prec):
    """A half request that fails in binary32 too (cond 1e10) ends as a binary64
    request does, beside others that fall back once, not at all, or start in
    binary32; every system is solved and counted once."""
    conds = [1e1, 1e10, 1e5, 1e10, 1e1, 1e5, 1e10]
    shapes = [(n, c, m) for n, c, m in zip((70, 90, 150, 257, 300, 410, 512), conds, (1, 2, 8, 3, 4, 1, 2))]
    _say("batched both fallbacks", prec)
    pb = spdgen.packed_batch(shapes, config=3, first_index=6100)
    asked = [prec] * 5 + ["fp32", "fp32"]
    _, X, r, p = _run(spd, pb, asked)
    _, X32, r32, p32 = _run(spd, pb, "fp32")
    _, X64, _, _ = _run(spd, pb, "fp64")
    assert np.all(r["status"] == 0), r
    assert list(p) == [spd.PREC[q] for q in (prec, "fp64", "fp32", "fp64", prec, "fp32", "fp64")], p
    assert list(r["fallbacks"]) == [0, 2, 1, 2, 0, 0, 1], r
    for s, (n, _, m) in enumerate(shapes):
        b = slice(int(pb.b_off[s]), int(pb.b_off[s]) + n * m)
        if p[s] == spd.PREC["fp64"]:
            assert np.array_equal(X[b], X64[b]), s
        elif p[s] == spd.PREC["fp32"]:
            assert np.array_equal(X[b], X32[b]), s


# the same in units of u cond
FORMER_ILL = {("fp32", 64): 0.1410, ("fp32", 128): 0.1219, ("fp64", 64): 0.1299, ("fp64", 128): 0.0921}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("top", [64, 128])
def test_first_solve_rounding_ill_conditioned(spd, prec, top):
    """As test_first_solve_rounding where elimination leaves little of A's
    values: cond 1e6, and 1e4 for binary32, whose factor still resolves that."""
    cond = 1e4 if prec == "fp32" else 1e6
    rng = np.random.Generator(np.random.PCG64(top + 1))
    pb = spdgen.packed_batch_grouped([(int(n), cond, 2) for n in rng.integers(top // 2, top + 1, 384)], seed=top + 1)
    pb.A, pb.B = pb.A.cpu().numpy(), pb.B.cpu().numpy()
    _, X, reps, _ = _run(spd, pb, prec, spd.default_opts(max_iter=0, fallback=0))
    err = []
    for s in range(384):
        n, a, b = int(pb.n[s]), int(pb.a_off[s]), int(pb.b_off[s])
        A, B = pb.A[a:a + n * n].reshape(n, n), pb.B[b:b + 2 * n].reshape(2, n).T
        x = np.linalg.solve(A, B)
        for _ in range(2):
            x = x + np.linalg.solve(A, (B - A.astype(np.longdouble) @ x).astype(np.float64))
        d = (X[b:b + 2 * n].reshape(2, n).T - x).astype(np.float64)
        err.append(np.linalg.norm(d) / np.linalg.norm(x.astype(np.float64)))
    err = float(np.exp(np.mean(np.log(err)))) / cond / (2.0 ** -24 if prec == "fp32" else 2.0 ** -53)
    _say(f"batched rounding, ill-conditioned {prec} n<={top}: {err:.4f}")
    assert err <= 1.05 * FORMER_ILL[prec, top], err
