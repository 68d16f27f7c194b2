"""A block of more than 32,767 nodes whose band is small enough for every step
to run in one launch: clusters of close frames at both ends and in the middle,
the other frames too far apart for any pair.  Equal to one launch per step and to
the trellis over the winning cluster alone, bit for bit."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,models", [(32767, 1), (32768, 2), (40000, 3)])
def test_one_launch_on_many_nodes(n, models):
    rng = np.random.Generator(np.random.PCG64(n))
    T, m = 5, 6
    step = np.full(n - 1, 2 * T, np.int64)
    for a in (0, n // 2, n - 101):
        step[a:a + 100] = 1
    t = np.concatenate([[0], np.cumsum(step)]).astype(np.int32)
    scene = synth.Points(rng.uniform(0, 40, (n, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, n, 8),
                         int(t[-1]) + 1)
    ms = []
    for q in range(models):
        mt = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m + q - 1))]).astype(np.int32)
        ms.append(synth.Points(rng.uniform(0, 40, (m + q, 2)).astype(np.float32), mt,
                               synth.dirichlet_desc(rng, m + q, 8)))
    p = synth.Params(T=T)
    ctx = stm.Context(0)
    a, b = stm.Trellis(ctx, ms, scene, p), stm.Trellis(ctx, ms, scene, p, stepwise=True)
    assert a.info()["fused"] and not b.info()["fused"] and a.info()["cells_per_step"] < 2000
    ra, rb = a.run(), b.run()
    assert np.isfinite(ra["energy32"]).all()
    for k in ("energy32", "energy64", "energy_u64", "assign"):
        np.testing.assert_array_equal(ra[k], rb[k])
    first = ra["assign"][0]  # the first model's optimum lies in one cluster
    lo = max(0, int(first) - 110)
    c = stm.Trellis(ctx, ms[:1], scene, p, lo, min(n, lo + 220))
    rc = c.run()
    assert rc["energy32"][0] == ra["energy32"][0]
    np.testing.assert_array_equal(c.model_rows(rc, 0), a.model_rows(ra, 0))
    for x in (a, b, c):
        x.close()
    ctx.close()
