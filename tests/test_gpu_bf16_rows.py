"""The BF16 unary table at the edges of its tiles: descriptor lengths around the
32 columns and row counts around the 16 rows a wave rounds at a time, the 16 x
64 tiles of the products and their padding, against FP64 distances of the
rounded descriptors."""
import numpy as np
import pytest
import torch

import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,dim", [(3, 1, 1), (3, 15, 31), (15, 16, 32), (16, 17, 33), (17, 63, 64), (33, 65, 96),
                                     (75, 257, 162), (5, 300, 256)])
def test_against_rounded_distances(m, n, dim):
    rng = np.random.Generator(np.random.PCG64(m * 1009 + n * 31 + dim))
    f, g = rng.uniform(-1, 1, (m, dim)).astype(np.float32), rng.uniform(-1, 1, (n, dim)).astype(np.float32)
    model = synth.Points(np.zeros((m, 2), np.float32), np.arange(m, dtype=np.int32), f)
    scene = synth.Points(np.zeros((n, 2), np.float32), np.zeros(n, np.int32), g, m + 1)
    p = synth.Params()
    p.unary_bf16 = True
    ctx = stm.Context(0)
    U = np.asarray(ctx.unary(model, scene, p), np.float64)
    ctx.close()
    fr, gr = (torch.from_numpy(x).to(torch.bfloat16).double().numpy() for x in (f, g))
    f2, g2, dot = (fr ** 2).sum(1), (gr ** 2).sum(1), fr @ gr.T
    d2 = f2[:, None] + g2[None, :] - 2 * dot
    # three sums of dim terms and their combination in FP32, one rounding each
    tol = (dim + 4) * 2.0 ** -24 * (f2[:, None] + g2[None, :] + 2 * (np.abs(fr) @ np.abs(gr).T))
    # the square root's own rounding on top
    assert (np.abs(U ** 2 - np.maximum(d2, 0)) <= tol + 2.0 ** -22 * np.maximum(d2, 0)).all()
