"""Launches by the number of matchings: few matchings take more working waves each
(short, medium and long lists) and four waves per re-score, many take fewer and
one.  A
range of offsets as one call equals its halves, quarters and single offsets bit
for bit on either side of every line, and the FP64 energies the oracle's of the
same assignments.  Short lists of few matchings keep their value tables in LDS:
models just inside and past its bound, longer than the 64 points a wave holds at a
time, coincident points and node-order causality, against the oracle."""
import numpy as np
import pytest

import oracle
from parity_check import check
import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,W,n_tau", [(16, 2, 1025), (16, 3, 2049), (8, 1, 4097), (32, 3, 513), (32, 2, 1025),
                                       (64, 3, 257)])
def test_parts_equal_whole(K, W, n_tau):
    rng = np.random.Generator(np.random.PCG64(K * 7 + W))
    m, per = 7, 8
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 60, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, 8))
    frames = n_tau + int(t[-1])
    st = np.repeat(np.arange(frames, dtype=np.int32), per)
    scene = synth.Points(rng.uniform(0, 60, (len(st), 2)).astype(np.float32), st,
                         synth.dirichlet_desc(rng, len(st), 8), frames)
    p = synth.Params(window=W, k_max=K, T=5)
    ctx = stm.Context(0)
    whole = ctx.match(model, scene, p, 0, n_tau)
    for parts in ([(0, n_tau // 2), (n_tau // 2, n_tau)], [(n_tau // 4, n_tau // 2)], [(0, n_tau - 1)],
                  [(3, 4), (n_tau - 1, n_tau)]):
        for b, e in parts:
            part = ctx.match(model, scene, p, b, e)
            np.testing.assert_array_equal(part["energy32"], whole["energy32"][b:e])
            np.testing.assert_array_equal(part["assign"], whole["assign"][b:e])
            np.testing.assert_allclose(part["energy64"], whole["energy64"][b:e], rtol=1e-12, atol=1e-12)
    rows = np.unique(np.linspace(0, n_tau - 1, 40).astype(int))
    fin = rows[np.isfinite(whole["energy32"][rows])]
    assert len(fin) > 10
    eg, _ = oracle.energies(model, scene, p, whole["assign"][fin])
    np.testing.assert_allclose(whole["energy64"][fin], eg, rtol=1e-9, atol=1e-9)
    ctx.close()


@pytest.mark.parametrize("m,K,W,per,grid,node", [
    (3, 16, 2, 5, 0, False), (46, 16, 2, 5, 0, False), (47, 16, 2, 5, 0, False), (10, 32, 2, 9, 0, False),
    (11, 32, 2, 9, 0, False), (130, 4, 1, 3, 0, False), (64, 8, 1, 4, 0, False), (12, 16, 2, 5, 15, False),
    (5, 1, 0, 2, 0, False), (12, 16, 2, 5, 0, True)])
def test_tables_in_lds(m, K, W, per, grid, node):
    rng = np.random.Generator(np.random.PCG64(m * 17 + K))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, m - 1))]).astype(np.int32)
    model = synth.Points(rng.uniform(0, 60, (m, 2)).astype(np.float32), t, synth.dirichlet_desc(rng, m, 8))
    frames = 21 + int(t[-1])
    st = np.repeat(np.arange(frames, dtype=np.int32), per)
    xy = rng.uniform(0, 60, (len(st), 2))
    xy = np.round(xy / grid) * grid if grid else xy
    scene = synth.Points(xy.astype(np.float32), st, synth.dirichlet_desc(rng, len(st), 8), frames)
    p = synth.Params(window=W, k_max=K, T=5)
    p.causal_node = node
    ctx = stm.Context(0)
    assert check(model, scene, p, ctx.match(model, scene, p), oracle.match(model, scene, p))["feasible"] > 0
    ctx.close()
