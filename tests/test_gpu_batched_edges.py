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
