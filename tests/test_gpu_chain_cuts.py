"""Chains of one call cut by the scratch limits: value tables past 4 GiB, so that
several chains run in more than one chunk of offsets (cut evenly or in full
chunks, whichever ends in fuller launches), and unary tables past 1 GiB, so that
chains go to several launches.  Every chain equals its lone matching bit for bit."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from oracle import chains as C
from parity_check import to_np
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,n_tau,per,n_chains,window", [
    (100, 1000, 20, 3, 3),   # two equal chunks
    (68, 1400, 20, 3, 3),    # a full chunk and a short one
    (50, 1400, 20, 4, 3),
    (90, 30, 12000, 3, 0)])  # 270 rows of a 1.2 GB table or more
def test_cut_calls_equal_lone_matchings(frames, n_tau, per, n_chains, window):
    rng = np.random.Generator(np.random.PCG64(frames + n_chains))
    t = np.concatenate([[0], np.cumsum(rng.integers(1, 3, frames - 1))]).astype(np.int32)
    mt = np.repeat(t, n_chains)
    n = len(mt)
    model = synth.Points(rng.uniform(0, 60, (n, 2)).astype(np.float32), mt, rng.random((n, 4), np.float32))
    F = n_tau + int(t[-1])
    st = np.repeat(np.arange(F, dtype=np.int32), per)
    scene = synth.Points(rng.uniform(0, 60, (len(st), 2)).astype(np.float32), st,
                         rng.random((len(st), 4), np.float32), F)
    tables = (frames - 2) * n_chains * n_tau * 64 * 64 * 4
    assert tables > 4 << 30 or n * len(st) * 4 > 1 << 30
    p = synth.Params(window=window, k_max=64, T=10)
    sal = rng.uniform(0, 1, n).astype(np.float32)
    ctx = stm.Context(0)
    ds = stm.DevicePoints.from_host(scene)
    got = ctx.match_chains(stm.DevicePoints.from_host(model), ds, p, sal, n_chains)
    assert len(got["energy32"]) == n_tau
    total = np.zeros(n_tau, np.float32)
    chains = C.build_chains(mt, sal, n_chains)
    assert len(chains) == n_chains
    for idx in chains:
        idx = np.asarray(idx)
        lone = ctx.match(stm.DevicePoints.from_host(C.sub_model(model, idx)), ds, p, 0, n_tau)
        np.testing.assert_array_equal(to_np(got["assign"])[:, idx], to_np(lone["assign"]))
        total += to_np(lone["energy32"])
    np.testing.assert_array_equal(to_np(got["energy32"]), total / np.float32(n_chains))
    assert np.isfinite(total).any()
    ctx.close()
