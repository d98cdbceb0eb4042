"""Activation of the sparse volume's blocks at the edges of its wavefronts (64
columns, groups of rows): images smaller than one, heights and widths one
beside a multiple, one to many scans, cubes of one block to several a side.
Against the oracle's activation as the other test of it: no block but the
oracle's at a radius 1e-7 m larger, every one of its blocks at a radius 1e-7 m
smaller, with first scans in order."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_sdf_hash import EPS, _export, _integrate, _key_map

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,n", [(2, 4, 1), (3, 63, 2), (4, 64, 1), (5, 65, 3), (15, 70, 1), (16, 256, 1),
                                   (17, 128, 5), (33, 130, 33), (64, 1000, 2)])
@pytest.mark.parametrize("radius", [0.0, 0.3, 4.1])
def test_activation_at_wavefront_edges(H, W, n, radius):
    import paper_2112_02779_amd as rir
    sm = synth.staggered_sensor(H, W, r0=0.02) if H % 2 else synth.uniform_sensor(H, W)
    rng = np.random.default_rng(1000 * H + W + n)
    ranges = (rng.uniform(1.0, 25.0, (n, H, W)) * (rng.random((n, H, W)) < 0.9)).astype(np.float32)
    ranges[:, H // 2] = rng.uniform(5.0, 5.5, (n, W))  # a row whose neighbours share cubes
    ranges[0, 0, 0], ranges[0, -1, -1] = np.nan, np.inf
    poses = np.stack([synth.inv_pose(synth.make_pose(synth.rot_axis_angle(synth.unit_vector(rng), 0.4 * k),
                                                     rng.uniform(-3, 3, 3))) for k in range(n)])
    vol = _integrate(rir, sm, ranges, poses, 0.3, 20.0, radius, max_blocks=60000, origin=(0.01, 0.02, 0.03))
    rows, _ = _export(vol)
    got = _key_map(rows)
    assert len(got) == len(rows) == vol.size()[0]
    inner = _key_map(oracle.sdf_activate(sm, ranges, poses, max(radius - EPS, 0.0), 20.0, 0.1, (0.01, 0.02, 0.03)))
    outer = _key_map(oracle.sdf_activate(sm, ranges, poses, radius + EPS, 20.0, 0.1, (0.01, 0.02, 0.03)))
    assert set(inner) <= set(got) <= set(outer), (len(set(inner) - set(got)), len(set(got) - set(outer)))
    for k, f in got.items():
        assert outer[k] <= f <= inner.get(k, 1 << 30), (k, f)
