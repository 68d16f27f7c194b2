"""The FP32 unary table at the edges of its tiles: model sizes around 16 R
rows, scene sizes around 16 and 64 points on both sides of the few-tiles rule,
descriptor lengths around the 32- and 64-dimension tiles.  The device sums in
FP32 in ascending order, so each entry is within (D + 2) roundings of 2^-24
relative of the FP64 distance."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = stm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("M,S,dim", [(3, 1, 1), (16, 16, 32), (17, 17, 33), (15, 63, 64), (33, 65, 65), (47, 130, 162),
                                     (81, 200, 256), (16, 8192, 5), (31, 8193, 32), (48, 8191, 31), (64, 8200, 63),
                                     (80, 8257, 162), (161, 4100, 161)])
def test_unary_at_tile_edges(ctx, M, S, dim):
    rng = np.random.Generator(np.random.PCG64(1000 * M + dim))
    model = synth.make_model(rng, M, 100.0, 100.0, 10, dim=dim)
    xy, t = rng.uniform(0, 100, (S, 2)).astype(np.float32), np.sort(rng.integers(0, 50, S)).astype(np.int32)
    scene = synth.Points(xy, t, rng.uniform(0, 1, (S, dim)).astype(np.float32), 50)
    U = ctx.unary(model, scene, synth.Params())
    f, g = model.desc.astype(np.float64), scene.desc.astype(np.float64)
    want = np.stack([np.sqrt(((g - row) ** 2).sum(1)) for row in f])
    assert U.shape == want.shape
    assert (np.abs(U - want) <= (dim + 2) * 2.0 ** -24 * want).all()
