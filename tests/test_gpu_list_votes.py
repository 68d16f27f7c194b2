"""Explicit lists around the rule that picks the variant for lists that repeat:
lists that change every two to five points or never, of a single offset and of
many, models of odd lengths.  Host and device lists and a plan's run take the
same rows bit for bit, and sampled rows the oracle's optimum."""
import numpy as np
import pytest

import oracle
import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth
from parity_check import to_np
from tolerances import energy_tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("every", [2, 3, 4, 5, 100])
@pytest.mark.parametrize("m,n", [(9, 1), (21, 90), (33, 40)])
def test_variants_agree(m, n, every):
    import torch
    rng = np.random.Generator(np.random.PCG64(m * 100 + every))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 40, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, 8))
    F, block = n + int(t[-1]), 40
    scene = synth.Points(rng.uniform(0, 40, (F + block, 2)).astype(np.float32),
                         np.minimum(np.arange(F + block), F - 1).astype(np.int32),
                         synth.dirichlet_desc(rng, F + block, 8), F)
    p = synth.Params(window=0, k_max=block, T=10)
    first = np.arange(n)[:, None] + np.minimum(np.arange(m) // every, 3)[None, :]
    cand = (first[:, :, None] + np.arange(block)).astype(np.int32)
    count = np.full((n, m), block, np.int32)
    ctx = stm.Context(0)
    host = ctx.match_lists(model, scene, p, cand, count, 0, n)
    dm, ds = stm.DevicePoints.from_host(model), stm.DevicePoints.from_host(scene)
    dc, dn = torch.as_tensor(cand, device="cuda"), torch.as_tensor(count, device="cuda")
    dev = ctx.match_lists(dm, ds, p, dc, dn, 0, n)
    plan = stm.Plan(ctx, [dm], [ds], [(0, 0)], p)
    assert plan.n_rows == n
    rows = plan.pair_rows(plan.run_lists([dc], [dn], block), 0)
    for k, got in zip(("energy32", "energy64", "energy_u64", "assign"), rows):
        np.testing.assert_array_equal(to_np(dev[k]), host[k])
        np.testing.assert_array_equal(to_np(got), host[k])
    pick = np.unique(np.linspace(0, n - 1, 5).astype(int))
    for b in pick:
        e = oracle.match_lists(model, scene, p, cand[b:b + 1], count[b:b + 1])["energy"]
        got = host["energy32"][b:b + 1]
        assert (np.isfinite(got) == np.isfinite(e)).all()
        if np.isfinite(e).all():
            assert (np.abs(got - e) <= energy_tol(e)).all()
    assert np.isfinite(host["energy32"]).any()
    plan.close()
    ctx.close()
