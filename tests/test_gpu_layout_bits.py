"""The same matching has the same bits in every layout of the recursion: short
lists in calls of few matchings (one barrier a step), of many (one wave a
matching) and in plans (the 64-slot layout), on scenes whose frames jump, so that
the frame terms are products that round."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from parity_check import to_np
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


def _pair(seed, m, n_tau):
    rng = np.random.Generator(np.random.PCG64(seed))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 8, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 60, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, 8))
    F = n_tau + int(t[-1])
    st = np.sort(rng.integers(0, F, F)).astype(np.int32)
    return model, synth.Points(rng.uniform(0, 60, (len(st), 2)).astype(np.float32), st,
                               synth.dirichlet_desc(rng, len(st), 8), F)


@pytest.mark.parametrize("m,K,W,extra", [
    (3, 12, 6, {}), (30, 12, 6, {}), (12, 16, 8, {}), (12, 17, 9, {}), (30, 32, 16, {}), (8, 4, 4, {}),
    (12, 16, 8, dict(closeness_span=True)), (12, 32, 16, dict(causal_node=True))])
def test_calls_and_plan(m, K, W, extra):
    n = 2200  # lists of at most 16: one wave a matching above 2048
    model, scene = _pair(100 * m + K, m, n)
    p = synth.Params(window=W, k_max=K, T=10, **extra)
    ctx = stm.Context(0)
    whole = ctx.match(model, scene, p, 0, n)
    fin = np.isfinite(whole["energy32"])
    assert fin.sum() > n // 8
    z = whole["assign"][fin]
    gap = np.abs(np.diff(model.t)[None, :] - np.diff(scene.t[z], axis=1))
    assert (gap > 2).any()  # some optima hold a term that is no power of two times l2
    for b, e in ((0, 200), (500, 900), (900, 2200)):
        part = ctx.match(model, scene, p, b, e)
        for k in ("energy32", "assign"):
            np.testing.assert_array_equal(part[k], whole[k][b:e], err_msg=f"{k} of [{b}, {e})")
    plan = stm.Plan(ctx, [model], [scene], [(0, 0)], p)
    e32, _, _, asg = plan.pair_rows(plan.run(), 0)
    np.testing.assert_array_equal(to_np(e32)[:n], whole["energy32"])
    np.testing.assert_array_equal(to_np(asg)[:n], whole["assign"])
    plan.close()
    ctx.close()
