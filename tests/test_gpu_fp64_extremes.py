"""FP64 registration with a kernel size so small that (e / delta)^2 overflows:
the pseudo-Huber weight 1 / sqrt(1 + (e / delta)^2) is then 0, not NaN, for
every residual but an exact zero, so the sums stay finite and no update is
made."""
import numpy as np
import pytest

import synth
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sensor", ["uniform", "staggered"])
def test_weight_of_overflowing_residuals(sensor):
    import torch
    import paper_2112_02779_amd as rir
    sm = synth.uniform_sensor(32, 512) if sensor == "uniform" else synth.staggered_sensor(32, 500, r0=0.015)
    pair = synth.gen_pair(synth.CONFIGS["pair64"], 3, sensor=sm)
    sen, ctx = rir.Sensor.from_model(sm), rir.Context(0)
    prm = rir.make_params(levels=2, iters=[2, 2], delta=1e-170, precision=1)
    src, dst = to_dev(pair.src), to_dev(pair.dst)
    out = rir.debug_associate(ctx, prm, sen, src, dst, 0, np.eye(4))
    w, e, mask = (out[k].cpu().numpy() for k in ("w", "e", "mask"))
    assert (mask == 1).sum() > 1000
    assert np.all(w[e != 0] == 0) and np.all(np.isfinite(w))
    for k in ("sum_w", "sum_w_e2", "robust_cost"):
        assert np.isfinite(out["stats"][k])
    assert np.all(np.isfinite(out["stats"]["JtJ"])) and np.all(np.isfinite(out["stats"]["Jtr"]))
    T, stats = rir.icp_batch(ctx, prm, [(sen, src, dst)])
    torch.cuda.synchronize()
    assert np.array_equal(T.cpu().numpy()[0], np.eye(4))
    st = rir.stats_to_numpy(stats, 1, 2)
    assert np.all(st["status"] != 0) and np.all(np.isfinite(st["sum_w"])) and np.all(np.isfinite(st["JtJ"]))
