"""Refused calls on device data: work that was queued before the inputs were
validated is over when the refusal is returned, and an invalid input or offset
range is reported as such also where the unary table could not be allocated."""
import numpy as np
import pytest

import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth

pytestmark = pytest.mark.gpu


def _outputs(n, m):
    import torch
    return dict(energy32=torch.empty(n, dtype=torch.float32, device="cuda"),
                energy64=torch.empty(n, dtype=torch.float64, device="cuda"),
                energy_u64=torch.empty(n, dtype=torch.float64, device="cuda"),
                assign=torch.empty((n, m), dtype=torch.int32, device="cuda"))


@pytest.mark.parametrize("past", [0, 1])
def test_refused_range_leaves_nothing_running(past):
    import torch
    rng = np.random.Generator(np.random.PCG64(5))
    m, F, per, dim = 400, 500, 600, 256
    model = synth.Points(rng.uniform(0, 60, (m, 2)).astype(np.float32), np.arange(m, dtype=np.int32),
                         rng.random((m, dim), np.float32))
    st = np.repeat(np.arange(F, dtype=np.int32), per)
    scene = synth.Points(rng.uniform(0, 60, (len(st), 2)).astype(np.float32), st,
                         rng.random((len(st), dim), np.float32), F)
    p = synth.Params(window=0, k_max=4, T=5)
    dm, ds = stm.DevicePoints.from_host(model), stm.DevicePoints.from_host(scene)
    ctx = stm.Context(0)
    ctx.match(dm, ds, p, 0, 2)  # the table is allocated
    out = _outputs(F + 1, m)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with pytest.raises(stm.StmError) as e:
            ctx.match(dm, ds, p, 0, F + past, out=out)  # past the last offset F - span
        assert stream.query()  # (the table takes milliseconds)
    assert e.value.code == stm.STM_EINVAL
    ctx.close()


def test_invalid_input_is_reported_before_memory():
    import torch
    n = 2_000_000  # the unary table would be 16 TB
    t = np.arange(n, dtype=np.int32)
    model = synth.Points(np.zeros((n, 2), np.float32), t, np.zeros((n, 1), np.float32))
    scene = synth.Points(np.zeros((n, 2), np.float32), t, np.zeros((n, 1), np.float32), n + 5)
    dm, ds = stm.DevicePoints.from_host(model), stm.DevicePoints.from_host(scene)
    p = synth.Params(window=0, k_max=4, T=5)
    ctx = stm.Context(0)
    out = _outputs(1, n)
    pr = stm.Pruner(ctx, 1)
    pr.set_params(synth.pruner_init(1, 0))
    group = np.zeros((1, 2), np.int32)
    for what, code in (("range", stm.STM_EINVAL), ("valid", stm.STM_ENOMEM), ("nan", stm.STM_EINVAL)):
        if what == "nan":
            dm.xy[n // 2, 0] = float("nan")
            torch.cuda.synchronize()
        b = 6 if what == "range" else 0  # n + 5 frames, a span of n - 1: offsets 0 .. 5
        with pytest.raises(stm.StmError) as e:
            ctx.match(dm, ds, p, b, b + 1, out=out)
        assert e.value.code == code, (what, str(e.value))
        if what != "range":
            with pytest.raises(stm.StmError) as e:
                pr.features(dm, ds, p, group)
            assert e.value.code == code, (what, str(e.value))
    pr.close()
    ctx.close()
