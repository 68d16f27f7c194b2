"""Step launches of 8 x 64 cells (many models on wide bands) with rows that have
only some of a tile's predecessors, row groups that are not full, a closeness
limit, both readings of it and coincident points: equal to lone models (4 x 64
cells) bit for bit, and sampled models to the FP64 oracle.  The tiling that a run
takes is told from its number of tiles."""
import numpy as np
import pytest

import oracle
import paper_1505_00581_amd as stm
from parity_check import check, to_np
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


def _tiles(t, T, rows):
    """Tiles of `rows` rows by 64 columns of a band of frames t that hold cells."""
    lo = np.searchsorted(t, t, "right")
    hi = np.searchsorted(t, t + T, "left") if T > 0 else np.full(len(t), len(t))
    hi = np.maximum(hi, lo)
    n = 0
    for r0 in range(0, len(t), rows):
        r1 = min(len(t), r0 + rows)
        for c0 in range(lo[r0], hi[r1 - 1], 64):
            c1 = min(hi[r1 - 1], c0 + 64)
            n += bool((np.minimum(hi[r0:r1], c1) - np.maximum(lo[r0:r1], c0)).clip(0).sum())
    return n, int((hi - lo).sum())


@pytest.mark.parametrize("n,per_frame,T,span,grid,models", [
    (403, 1, 0, False, 0, 60), (403, 5, 0, False, 0, 60), (401, 7, 0, True, 0, 60), (390, 13, 0, False, 8, 60),
    (506, 5, 60, False, 0, 60), (506, 5, 60, True, 8, 60), (755, 3, 100, False, 0, 25)])
def test_tall_tiles(n, per_frame, T, span, grid, models):
    rng = np.random.Generator(np.random.PCG64(n * 3 + per_frame))
    xy = rng.uniform(0, 40, (n, 2))
    xy = np.round(xy / grid) * grid if grid else xy
    t = (np.arange(n) // per_frame).astype(np.int32)
    scene = synth.Points(xy.astype(np.float32), t, synth.dirichlet_desc(rng, n, 8), int(t[-1]) + 1)
    ms = []
    for q in range(models):
        mt = np.concatenate([[0], np.cumsum(rng.integers(1, 3, 4))]).astype(np.int32)
        ms.append(synth.Points(rng.uniform(0, 40, (5, 2)).astype(np.float32), mt, synth.dirichlet_desc(rng, 5, 8)))
    p = synth.Params(T=T, closeness_span=span)
    tall, cells = _tiles(t, T, 8)
    flat, _ = _tiles(t, T, 4)
    assert cells >= 128 * n and tall * models >= 8192 and tall < flat  # the rule for 8 x 64 cells
    ctx = stm.Context(0)
    many = stm.Trellis(ctx, ms, scene, p, stepwise=True)
    assert many.info()["tiles"] == tall and many.info()["degenerate"] == bool(grid)
    out = many.run()
    for q in (0, models // 2, models - 1):
        one = stm.Trellis(ctx, [ms[q]], scene, p, stepwise=True)
        assert one.info()["tiles"] == flat
        r = one.run()
        for k in ("energy32", "energy64", "energy_u64"):
            assert to_np(out[k])[q] == to_np(r[k])[0], (k, q)
        np.testing.assert_array_equal(to_np(many.model_rows(out, q)), to_np(one.model_rows(r, 0)))
        one.close()
    row = dict(energy32=to_np(out["energy32"])[:1], energy64=to_np(out["energy64"])[:1],
               energy_u64=to_np(out["energy_u64"])[:1], assign=to_np(many.model_rows(out, 0))[None, :])
    check(ms[0], scene, p, row, oracle.match_trellis(ms[0], scene, p))
    many.close()
    ctx.close()
