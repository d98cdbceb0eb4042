"""Re-projection under per-column poses where its launches and workgroups end:
more scans than a launch takes, a column block that is not full, rows that do
not divide by the rows of a workgroup, and rotations on both sides of one
radian (the two forms of the column's pose).  Against the FP64 oracle as the
other tests of this operation."""
import numpy as np
import pytest

import synth
from parity_util import to_dev
from test_gpu_deskew import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,H,W,n", [("uniform", 9, 66, 67), ("uniform", 33, 128, 3), ("staggered", 35, 100, 65)])
def test_deskew_launch_edges(kind, H, W, n):
    import paper_2112_02779_amd as rir
    sm = synth.uniform_sensor(H, W) if kind == "uniform" else synth.staggered_sensor(H, W, r0=0.02)
    rng = np.random.default_rng(H * W + n)
    imgs = (rng.uniform(4.0, 30.0, (n, H, W)) * (rng.random((n, H, W)) < 0.9)).astype(np.float32)
    xi = rng.uniform(-0.3, 0.3, (n, 6))
    xi[0] = 0.0
    xi[1, :3] = (0.1, -0.2, 3.0)     # 1.5 rad at the image's ends
    xi[n - 1, :3] = (0.0, 0.0, 1.0)
    out = rir.deskew(rir.Sensor.from_model(sm), to_dev(imgs), xi).cpu().numpy()
    for k in (0, 1, 2, n // 2, n - 2, n - 1):
        check(sm, imgs[k], xi[k], out[k])
