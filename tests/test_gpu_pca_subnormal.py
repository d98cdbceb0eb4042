"""PCA normals of subnormal ranges, where the FP32 limit of the window's range
test has few bits: the same points take part as in the image scaled up by a
power of two, whose decisions are the same in FP64."""
import numpy as np
import pytest

import synth
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [1, 2])
def test_range_test_of_subnormal_ranges(half):
    import paper_2112_02779_amd as rir
    # beams far apart: the points' spread is that of their ranges, and its
    # fourth power is still a double
    sen = rir.Sensor.from_model(synth.uniform_sensor(16, 8, fov_up_deg=80.0, fov_down_deg=-80.0))
    rng = np.random.default_rng(4)
    # 0.1 x 713636 = 71363.6: one neighbour 71363 away is in, 71364 is not
    k = rng.choice([713636, 713636 + 71363, 713636 + 71364, 713636 - 71364], size=(16, 8))
    small = np.ldexp(k.astype(np.float64), -149).astype(np.float32)
    assert np.array_equal(np.ldexp(small.astype(np.float64), 149), k)
    valid = [rir.normals_pca(sen, to_dev(img), half=half, edge_rel=0.1)[1].cpu().numpy()
             for img in (k.astype(np.float32), small)]
    assert 0 < valid[0].sum() < valid[0].size
    np.testing.assert_array_equal(valid[1], valid[0])
