"""Trellis step launches of 4 x 64 and 8 x 64 cells with the operands in
registers, at the edges of their tiles: blocks of a few nodes, around one and
two column windows and row groups that are not full, several points per frame
(predecessors of some rows only), both readings of closeness and coincident
points, against the FP64 oracle; many models (8 x 64) equal to lone ones
(4 x 64) bit for bit; backtracking on more nodes than it holds in LDS; and
every step in one launch, with a model's columns cut into 16, 8 or 1 parts and
models of different sizes, equal to one launch per step bit for bit."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_1505_00581_amd as stm
from parity_check import check, to_np
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = stm.Context(0)
    yield c
    c.close()


def _block(seed, n, per_frame, m=5, grid=0):
    """A model of m points and a scene of n nodes, per_frame of them in each frame."""
    rng = np.random.Generator(np.random.PCG64(seed))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 40, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, 8))
    xy = rng.uniform(0, 40, (n, 2))
    if grid:
        xy = np.round(xy / grid) * grid
    st = (np.arange(n) // per_frame).astype(np.int32)
    return model, synth.Points(xy.astype(np.float32), st, synth.dirichlet_desc(rng, n, 8), int(st[-1]) + 1)


def _rows(tr, out, q):
    return dict(energy32=to_np(out["energy32"])[q:q + 1], energy64=to_np(out["energy64"])[q:q + 1],
                energy_u64=to_np(out["energy_u64"])[q:q + 1], assign=to_np(tr.model_rows(out, q))[None, :])


@pytest.mark.parametrize("n,per_frame,T,span,grid", [
    (5, 1, 0, False, 0), (6, 1, 3, False, 0), (9, 2, 0, False, 0), (63, 1, 0, False, 0), (64, 1, 0, True, 0),
    (65, 1, 0, False, 0), (66, 3, 0, False, 0), (68, 1, 40, False, 0), (70, 5, 6, False, 0), (71, 5, 6, True, 0),
    (72, 7, 4, False, 10), (129, 1, 0, False, 0), (131, 4, 9, True, 10), (131, 30, 3, False, 0)])
def test_wide_tiles_against_oracle(ctx, n, per_frame, T, span, grid):
    m, s = _block(9000 + n, n, per_frame, grid=grid)
    p = synth.Params(T=T, closeness_span=span)
    tr = stm.Trellis(ctx, [m], s, p, stepwise=True)
    out = tr.run()
    check(m, s, p, _rows(tr, out, 0), oracle.match_trellis(m, s, p))
    assert not tr.info()["fused"]
    tr.close()


@pytest.mark.parametrize("n,per_frame,T,models", [(403, 1, 0, 700), (150, 25, 4, 500), (130, 2, 0, 600)])
def test_tall_tiles_equal_flat_ones(ctx, n, per_frame, T, models):
    pairs = [_block(9500 + q, n, per_frame, m=4) for q in range(3)]
    s = pairs[0][1]
    ms = [pairs[q % 3][0] for q in range(models)]
    p = synth.Params(T=T)
    many = stm.Trellis(ctx, ms, s, p, stepwise=True)
    out = many.run()
    for q in range(3):
        one = stm.Trellis(ctx, [ms[q]], s, p, stepwise=True)
        r = one.run()
        assert one.info()["tiles"] > many.info()["tiles"]
        for at in (q, models - 3 + (q - models) % 3):
            assert to_np(out["energy32"])[at] == to_np(r["energy32"])[0]
            assert to_np(out["energy64"])[at] == to_np(r["energy64"])[0]
            np.testing.assert_array_equal(to_np(many.model_rows(out, at)), to_np(one.model_rows(r, 0)))
        one.close()
    many.close()


@pytest.mark.parametrize("n", [4096, 4097, 4400])
def test_backtracking_on_many_nodes(ctx, n):
    # past node 4000 the frames lie T apart, so no path goes there: the optimum
    # is that of the first 4000 nodes
    m, s = _block(9900, n, 2, m=6)
    p = dataclasses.replace(synth.Params(T=4))
    t = s.t.copy()
    t[4000:] = t[3999] + 4 * (1 + np.arange(n - 4000))
    s = synth.Points(s.xy, t.astype(np.int32), s.desc, int(t[-1]) + 1)
    a, b = stm.Trellis(ctx, [m], s, p), stm.Trellis(ctx, [m], s, p, 0, 4000)
    ra, rb = a.run(), b.run()
    assert np.isfinite(ra["energy32"]).all()
    for k in ("energy32", "energy64", "energy_u64", "assign"):
        np.testing.assert_array_equal(ra[k], rb[k])
    a.close()
    b.close()


@pytest.mark.parametrize("n,per_frame,T,span,grid,models", [
    (5, 1, 3, False, 0, 1), (17, 1, 3, False, 0, 2), (200, 1, 10, False, 0, 1), (200, 1, 10, True, 0, 30),
    (201, 3, 4, False, 10, 3), (150, 1, 0, False, 0, 1), (127, 1, 0, False, 0, 2), (400, 2, 5, False, 0, 257)])
def test_column_parts_equal_step_launches(ctx, n, per_frame, T, span, grid, models):
    s = _block(9700 + n, n, per_frame, grid=grid)[1]
    ms = [_block(9700 + n + q, n, per_frame, m=3 + q % 7)[0] for q in range(models)]
    p = synth.Params(T=T, closeness_span=span)
    a, b = stm.Trellis(ctx, ms, s, p), stm.Trellis(ctx, ms, s, p, stepwise=True)
    ra, rb = a.run(), b.run()
    assert a.info()["fused"] == (a.info()["cells_per_step"] <= 8192) and not b.info()["fused"]
    for k in ("energy32", "energy64", "energy_u64", "assign"):
        np.testing.assert_array_equal(ra[k], rb[k])
    a.close()
    b.close()
