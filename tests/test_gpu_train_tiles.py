"""The training pass at the edges of its tiles: descriptor lengths around the
32-input tiles of layer 1 and the 64-column tiles of the weight gradients, odd
lengths, group counts around the chunk rule (64 ceil(G / 128) rows) and empty
slots, against the FP64 oracle with the rounding bounds of its sums."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from oracle import pruner as PR
from paper_1505_00581_amd import synth
from test_gpu_pruner import H, _gradient_magnitudes, _labelled, oracle_rows, random_groups, unpack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = stm.Context(0)
    yield c
    c.close()


def _inputs(dim, k_max):
    rng = np.random.Generator(np.random.PCG64(dim))
    p = synth.Params(window=2, k_max=k_max)
    model = synth.make_model(rng, 9, 160.0, 120.0, p.T, frame_hi=13, dim=dim)
    scene, _ = synth.make_scene(rng, [model], 40, np.full(40, 4), 160.0, 120.0, 1)
    return model, scene, p


@pytest.mark.parametrize("dim,n_groups,k_max", [(1, 3, 16), (8, 2, 20), (31, 2, 5), (32, 2, 16), (33, 5, 20),
                                                (56, 2, 16), (57, 2, 16), (63, 2, 16), (64, 3, 16), (65, 2, 16),
                                                (162, 127, 16), (162, 129, 20), (255, 2, 16), (256, 2, 16)])
def test_gradient_at_tile_edges(ctx, dim, n_groups, k_max):
    model, scene, p = _inputs(dim, k_max)
    pr = stm.Pruner(ctx, dim)
    theta = synth.pruner_init(dim, 3)
    pr.set_params(theta)
    groups = random_groups(model, scene, n_groups, seed=4)
    node, phi, q = pr.features(model, scene, p, groups)
    labels, slots = _labelled(model, scene, node, 6)
    loss, grad, scores = pr.gradient(model, scene, p, groups, labels)
    X, valid = oracle_rows(model, scene, p, groups, node, q)
    X[:, 2 * dim:] = phi.reshape(-1, 8)  # the pass is judged on the features it read (tested on their own)
    P = unpack(theta.astype(np.float64), dim)
    s, cache = PR.forward(P, X)
    want_loss, ds = PR.group_loss(s.reshape(-1, 64), None, slots, valid)
    g = PR.backward(P, cache, ds.reshape(-1))
    assert abs(loss - want_loss) <= 1e-4 * max(1.0, abs(want_loss))
    sv = s.reshape(-1, 64)[valid]
    assert (np.abs(scores[valid] - sv) <= 1e-4 * (1 + np.abs(sv))).all()
    assert np.isneginf(scores[~valid]).all()
    G = unpack(grad, dim)
    mag, extra = _gradient_magnitudes(P, cache, ds.reshape(-1))
    n_chain = X.shape[0] + 2 * (2 * dim + 8) + 2 * H  # longest chain of additions behind an element
    for k in P:
        tol = 1e-3 * np.abs(g[k]) + n_chain * 2.0 ** -24 * mag[k] + extra[k]
        assert (np.abs(G[k] - g[k]) <= tol).all(), k
    pr.close()
