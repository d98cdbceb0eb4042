"""Zero crossings of noise volumes, where every bit of the rows' masks and of
the three neighbour planes takes part: single blocks, rows of blocks along each
axis (their number no multiple of eight), with and without the jump test.  The
same FP32 values on both sides, so the same count, and every point within the
FP32 rounding of its coordinates (below 8 m: 4.8e-7 each)."""
import numpy as np
import pytest

import oracle
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [(1, 1, 1), (9, 1, 1), (1, 9, 1), (1, 1, 9), (2, 3, 2)])
@pytest.mark.parametrize("max_jump", [0.3, np.inf])
def test_extract_of_noise(nb, max_jump):
    from scipy.spatial import cKDTree
    import paper_2112_02779_amd as rir
    vol = rir.Volume(nb, (-1.0, -0.5, 0.25), 0.05)
    rng = np.random.default_rng(sum(nb))
    shape = (16 * nb[2], 16 * nb[1], 16 * nb[0])
    s = rng.uniform(-0.3, 0.3, shape).astype(np.float32)
    s[rng.random(shape) < 0.1] = 0.0
    w = (rng.random(shape) < 0.8).astype(np.float32)
    blocks = np.stack([s, w], -1).reshape(nb[2], 16, nb[1], 16, nb[0], 16, 2).transpose(0, 2, 4, 1, 3, 5, 6)
    got, n = rir.sdf_extract(vol, to_dev(np.ascontiguousarray(blocks)), min_weight=1.0, max_jump=max_jump)
    got = got.cpu().numpy().astype(np.float64)
    ref = oracle.sdf_extract(vol.origin, vol.voxel, s.astype(np.float64), w.astype(np.float64), 1.0, max_jump)
    assert n == len(ref) == len(got) and n > 1000
    d1, _ = cKDTree(ref).query(got)
    d2, _ = cKDTree(got).query(ref)
    assert d1.max() < 1e-6 and d2.max() < 1e-6, (d1.max(), d2.max())
