"""Explicit lists that stay the same for several points (blocks searched whole):
the recursion keeps the schedule, the cells and the directions of a step over
such runs.  Runs of every length against the FP64 oracle: one list for all
points, lists that move on after a few points, alternate, repeat with fewer
nodes or change at every point; one, two and more chunks a wave (short and long
closeness limits, none), models longer than the 64 points a wave holds at a time,
the span reading and coincident points; the plan's run equal to the per-model
run bit for bit."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_1505_00581_amd as stm
from oracle import energy as E
from paper_1505_00581_amd import synth
from tolerances import energy_tol

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = stm.Context(0)
    yield c
    c.close()


def _case(seed, m, n, per_frame, grid):
    """A model of m points and a sparse scene of n nodes (at most per_frame in a frame)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 40, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, 8))
    xy = rng.uniform(0, 40, (n, 2))
    if grid:
        xy = np.round(xy / grid) * grid
    st = (np.cumsum(rng.integers(0, 2, n)) if per_frame > 1 else np.arange(n)).astype(np.int32)
    frames = max(int(st[-1]) + 1, int(t[-1]) + 4)
    return model, synth.Points(xy.astype(np.float32), st, synth.dirichlet_desc(rng, n, 8), frames)


def _lists(pattern, rows, m, n, block):
    cand = np.zeros((rows, m, block), np.int32)
    count = np.full((rows, m), block, np.int32)
    j = np.arange(m)
    lo = {"same": 0 * j, "moves": 3 * (j // 5), "alternates": 2 * (j % 2), "fewer": 0 * j, "every": j}[pattern]
    for b in range(rows):
        cand[b] = np.minimum(lo + b, n - block)[:, None] + np.arange(block)
    if pattern == "fewer":
        count[:, m // 2:] = max(1, block - 3)
    return cand, count


@pytest.mark.parametrize("m,block,T,pattern,per_frame,span,grid", [
    (3, 60, 10, "same", 1, False, 0), (4, 60, 10, "same", 2, False, 0), (5, 64, 10, "same", 1, False, 0),
    (20, 60, 10, "same", 1, False, 0), (20, 60, 4, "same", 2, False, 0), (20, 64, 17, "same", 1, False, 0),
    (12, 64, 0, "same", 1, False, 0), (12, 33, 3, "same", 2, False, 0), (20, 60, 10, "same", 2, True, 0),
    (12, 60, 10, "same", 2, False, 10), (75, 64, 10, "moves", 1, False, 0), (75, 40, 6, "moves", 2, False, 0),
    (20, 64, 0, "moves", 1, False, 0), (20, 60, 10, "alternates", 1, False, 0), (20, 60, 10, "fewer", 1, False, 0),
    (20, 64, 17, "fewer", 2, False, 0), (20, 60, 10, "every", 1, False, 0)])
def test_runs_against_oracle(ctx, m, block, T, pattern, per_frame, span, grid):
    import torch
    model, scene = _case(m * 131 + block * 7 + T + per_frame, m, 190, per_frame, grid)
    p = synth.Params(window=0, k_max=block, T=T)
    p = dataclasses.replace(p, closeness_span=span) if span else p
    rows = min(6, len(E.offsets(model.t, scene.n_frames)))
    cand, count = _lists(pattern, rows, m, scene.n, block)
    got = ctx.match_lists(model, scene, p, cand, count, 0, rows)
    ora = oracle.match_lists(model, scene, p, cand, count)
    e = ora["energy"]
    fin = np.isfinite(e)
    np.testing.assert_array_equal(np.isfinite(got["energy32"]), fin)
    assert (np.abs(got["energy32"][fin] - e[fin]) <= energy_tol(e[fin])).all()
    if fin.any():  # the assignment is optimal, and made of listed nodes
        eg, _ = oracle.energies(model, scene, p, got["assign"][fin])
        assert (np.abs(eg - e[fin]) <= energy_tol(e[fin])).all()
        np.testing.assert_allclose(got["energy64"][fin], eg, rtol=1e-9, atol=1e-9)

    ds, dm = stm.DevicePoints.from_host(scene), stm.DevicePoints.from_host(model)
    plan = stm.Plan(ctx, [dm], [ds], np.zeros((1, 2), np.int32), p)
    n = int(plan.row_offsets[1])
    pc, pn = np.zeros((n, m, block), np.int32), np.zeros((n, m), np.int32)
    pc[:rows], pn[:rows] = cand, count
    out = plan.run_lists([torch.as_tensor(pc, device="cuda")], [torch.as_tensor(pn, device="cuda")], block)
    e32, e64, _, A = [x.cpu().numpy() for x in plan.pair_rows(out, 0)]
    np.testing.assert_array_equal(e32[:rows], got["energy32"])
    np.testing.assert_array_equal(A[:rows], got["assign"])
    assert not np.isfinite(e32[rows:]).any()
    plan.close()
