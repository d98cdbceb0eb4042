"""The counts inside a tile's record: 16 bits each, 4096 pixels in the largest
tile a tuning gives.  Scans without a gap, where nearly every pixel counts, give
the same counts and poses whatever the tile (the poses up to the rounding of
sums taken in another order)."""
import numpy as np
import pytest

import synth
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("solve_in_step", [0, 1])
def test_counts_of_the_largest_tile(prec, solve_in_step):
    import paper_2112_02779_amd as rir
    sm = synth.uniform_sensor(64, 1024)
    r = (10.0 + np.cos(2 * np.pi * np.arange(1024) / 1024))[None, :] * np.ones((64, 1))
    src, dst = to_dev(r.astype(np.float32)), to_dev((r + 0.01).astype(np.float32))
    sen = rir.Sensor.from_model(sm)
    prm = rir.make_params(levels=1, iters=[1], delta=0.5, precision=prec)
    got = []
    for block, px in ((64, 1), (256, 16), (256, 8)):
        ctx = rir.Context(0)
        ctx.set_tuning(block=block, px_per_thread=px, solve_in_step=solve_in_step)
        T, st = rir.icp_batch(ctx, prm, [(sen, src, dst)])
        got.append((T.cpu().numpy()[0], rir.stats_to_numpy(st, 1, 1)[0, 0]))
    for T, st in got:
        assert [st[k] for k in ("n_proj", "n_valid", "n_inlier")] == \
            [got[0][1][k] for k in ("n_proj", "n_valid", "n_inlier")]
        assert np.abs(T - got[0][0]).max() < 1e-6
    assert got[0][1]["n_proj"] == 64 * 1024 and got[0][1]["n_valid"] == got[0][1]["n_inlier"] == 62 * 1024
