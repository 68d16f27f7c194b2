"""Sums of the weight gradients over large batches: 65,536 times one group, whose
mean gradient is that of the group alone (the scale is a power of two), so that
only the rounding of the sums over the batch is left.  Each element is held to
the a-priori bound of chains of 512 rows and eight sums of their partial sums,
u times the sum of the magnitudes of all intermediate sums."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from oracle import pruner as PR
from paper_1505_00581_amd import synth
from test_gpu_pruner import oracle_rows, unpack

pytestmark = pytest.mark.gpu

CHAIN, LANES = 512, 8


def _bound(terms, repeats):
    """u x the sum of |intermediate sums| of terms [R, ...] repeated: chains of
    CHAIN terms, then LANES sums of the chains and three joins; and of the one
    repetition that is the reference."""
    u = 2.0 ** -24
    acc, mag, one = np.zeros(terms.shape[1:]), np.zeros(terms.shape[1:]), 0.0
    for r in range(CHAIN):
        acc = acc + terms[r % len(terms)]
        mag += np.abs(acc)
        if r == len(terms) - 1:
            one = mag.copy()
    chains = repeats * len(terms) // CHAIN
    per_lane = chains // LANES
    reduce = LANES * per_lane * (per_lane + 1) / 2 * np.abs(acc)
    return 1.05 * u * (mag * chains + reduce + 3 * chains * np.abs(acc) + one * repeats)


def test_weight_gradients_of_a_large_batch():
    dim, G = 8, 65536
    rng = np.random.Generator(np.random.PCG64(11))
    model = synth.make_model(rng, 9, 160.0, 120.0, 10, frame_hi=13, dim=dim)
    scene, _ = synth.make_scene(rng, [model], 40, np.full(40, 16), 160.0, 120.0, 1)
    p = synth.Params(window=2, k_max=64)
    ctx = stm.Context(0)
    pr = stm.Pruner(ctx, dim)
    theta = synth.pruner_init(dim, 3)
    pr.set_params(theta)
    group = np.array([[4, 5]], np.int32)
    node, phi, q = pr.features(model, scene, p, group)
    label = node[:, 7].copy()
    assert label[0] >= 0
    loss1, grad1, _ = pr.gradient(model, scene, p, group, label)
    loss, grad, _ = pr.gradient(model, scene, p, np.repeat(group, G, 0), np.repeat(label, G))
    assert abs(loss - loss1) <= 1e-6 * abs(loss1)
    # the group's terms in 64 bits
    X, valid = oracle_rows(model, scene, p, group, node, q)
    P = unpack(theta.astype(np.float64), dim)
    s, (X, h1, h2) = PR.forward(P, X)
    _, ds = PR.group_loss(s.reshape(-1, 64), None, np.array([7]), valid)
    dz2 = np.outer(ds.reshape(-1), P["w3"]) * (h2 > 0)
    dz1 = (dz2 @ P["W2"]) * (h1 > 0)
    got, one = unpack(grad, dim), unpack(grad1, dim)
    for name, terms, a, b in (
            ("W2", dz2[:, :, None] * h1[:, None, :], got["W2"], one["W2"]),
            ("W1 scene half", dz1[:, :, None] * X[:, None, dim:], got["W1"][:, dim:], one["W1"][:, dim:]),
            ("W1 model half", (dz1.sum(0)[:, None] * X[0, None, :dim])[None], got["W1"][:, :dim], one["W1"][:, :dim])):
        bound = _bound(terms, G) / G
        err = np.abs(a.astype(np.float64) - b.astype(np.float64))
        print(f"{name}: largest error {np.max(err / np.maximum(bound, 1e-300)):.3f} of its bound")
        assert (err <= bound).all(), name
    pr.close()
    ctx.close()
