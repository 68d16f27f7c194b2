"""Chains of a model solved in one launch, four at a time: one, four, five and
nine chains equal their lone matchings bit for bit, with lists of every layout
(short, medium, long), dummies, unsigned angles and a sparse scene."""
import dataclasses

import numpy as np
import pytest

import paper_1505_00581_amd as stm
from oracle import chains as C
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chains,K,W,per,extra", [
    (1, 64, 3, 14, {}), (4, 16, 2, 5, {}), (5, 32, 2, 9, {}), (9, 64, 2, 14, {}), (5, 64, 12, 2, {}),
    (5, 64, 2, 12, dict(w_dummy=0.5)), (5, 64, 2, 12, dict(angle_unsigned=True))])
def test_parts_equal_lone_matchings(n_chains, K, W, per, extra):
    rng = np.random.Generator(np.random.PCG64(n_chains * 100 + K + W))
    frames = np.cumsum(rng.integers(1, 3, 8)).astype(np.int32)
    mt = np.repeat(frames - frames[0], n_chains)  # every chain as long as the frames
    mt = np.delete(mt, np.nonzero(mt == mt[0])[0][-1]) if n_chains > 1 else mt  # but the last
    n = len(mt)
    model = synth.Points(rng.uniform(0, 60, (n, 2)).astype(np.float32), mt, synth.dirichlet_desc(rng, n, 8))
    F = 80
    st = np.repeat(np.arange(F, dtype=np.int32), per)
    scene = synth.Points(rng.uniform(0, 60, (len(st), 2)).astype(np.float32), st,
                         synth.dirichlet_desc(rng, len(st), 8), F)
    p = synth.Params(window=W, k_max=K, T=6)
    for k, v in extra.items():
        setattr(p, k, v)
    sal = rng.uniform(0, 1, n).astype(np.float32)
    ctx = stm.Context(0)
    got = ctx.match_chains(model, scene, p, sal, n_chains)
    n_tau = len(got["energy32"])
    total = np.zeros(n_tau, np.float32)
    chains = [c for c in C.build_chains(mt, sal, n_chains) if len(c) >= 3]
    for idx in chains:
        idx = np.asarray(idx)
        d = int(mt[idx[0]] - mt[0])
        lone = ctx.match(C.sub_model(model, idx), scene, p, d, d + n_tau)
        np.testing.assert_array_equal(got["assign"][:, idx], lone["assign"])
        total += lone["energy32"]
    np.testing.assert_array_equal(got["energy32"], total / np.float32(len(chains)))
    assert np.isfinite(total).any()
    ctx.close()
