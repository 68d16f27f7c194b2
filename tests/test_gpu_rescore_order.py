"""FP64 energies do not depend on how many matchings a launch re-scores: a call
or a plan of more than 2048 rows (one wave a matching) equals calls of a few
rows (four waves) bit for bit, for models of less than a wave, of several waves
and of more points than are summed at a time, with dummies and unsigned angles."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from parity_check import to_np
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


def _pair(seed, m, n_tau, dim=20):
    rng = np.random.Generator(np.random.PCG64(seed))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 60, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, dim))
    st = np.repeat(np.arange(n_tau + int(t[-1]), dtype=np.int32), 3)
    return model, synth.Points(rng.uniform(0, 60, (len(st), 2)).astype(np.float32), st,
                               synth.dirichlet_desc(rng, len(st), dim), n_tau + int(t[-1]))


@pytest.mark.parametrize("m,extra", [(3, {}), (75, {}), (257, {}), (300, {}), (70, dict(w_dummy=0.2)),
                                     (70, dict(angle_unsigned=True)), (260, dict(w_dummy=0.2))])
def test_calls_of_many_and_few_rows(m, extra):
    n = 4097  # one wave a matching above 2048
    model, scene = _pair(m, m, n)
    p = synth.Params(window=1, k_max=8, T=5, **extra)
    ctx = stm.Context(0)
    whole = ctx.match(model, scene, p, 0, n)
    assert np.isfinite(whole["energy64"]).sum() > n // 2
    for b, e in ((0, 300), (2000, 2001), (n - 200, n)):
        part = ctx.match(model, scene, p, b, e)
        for k in ("energy64", "energy_u64", "energy32", "assign"):
            np.testing.assert_array_equal(part[k], whole[k][b:e], err_msg=k)
    ctx.close()


def test_plan_rows_equal_calls():
    pairs = [_pair(s, m, 1500) for s, m in ((1, 20), (2, 66), (3, 130))]
    p = synth.Params(window=1, k_max=8, T=5)
    ctx = stm.Context(0)
    plan = stm.Plan(ctx, [m for m, _ in pairs], [s for _, s in pairs], [(q, q) for q in range(3)], p)
    out = plan.run()
    assert plan.n_rows > 4096
    for q, (model, scene) in enumerate(pairs):
        one = ctx.match(model, scene, p)
        e32, e64, eu, asg = plan.pair_rows(out, q)
        for got, k in ((e32, "energy32"), (e64, "energy64"), (eu, "energy_u64"), (asg, "assign")):
            np.testing.assert_array_equal(to_np(got), one[k], err_msg=k)
    plan.close()
    ctx.close()
