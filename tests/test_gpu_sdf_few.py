"""The forms of SDF fusion: layers with tile maxima, layers without (a stream
under capture, more than 2048 blocks, more than 3 scans, no receiver offset),
columns without (fewer blocks, fewer scans or a receiver offset).  The volumes
are equal to the last bit, and so is a smaller volume (2028 blocks) with the
part of the larger one (2197 blocks) that it covers."""
import numpy as np
import pytest
import torch

import synth
from parity_util import to_dev
import paper_2112_02779_amd as rir
from test_gpu_sdf import sequence

pytestmark = pytest.mark.gpu


def _captured(sen, vol, scans, poses, trunc, clip):
    vox = vol.alloc()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rir.sdf_integrate(sen, vol, vox, scans, poses, trunc, clip)
    graph.replay()
    torch.cuda.synchronize()
    return vox


@pytest.mark.parametrize("sensor", ["uniform", "uniform, odd width", "staggered"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("trunc,clip", [(0.3, 12.0), (0.0, 0.0)])
def test_forms_agree(sensor, n, trunc, clip):
    sm = {"uniform": lambda: synth.uniform_sensor(32, 512), "uniform, odd width": lambda: synth.uniform_sensor(32, 333),
          "staggered": lambda: synth.staggered_sensor(32, 500, r0=0.02)}[sensor]()
    sen = rir.Sensor.from_model(sm)
    ranges, poses, seq = sequence(sm, n, seed=8)
    scans, c = to_dev(ranges), seq["poses"][n // 2][:3, 3]
    origin = (c[0] - 10.4, c[1] - 10.4, -1.0)
    big, small = rir.Volume((13, 13, 13), origin, 0.1), rir.Volume((13, 13, 12), origin, 0.1)
    tiled = big.alloc()
    rir.sdf_integrate(sen, big, tiled, scans, poses, trunc, clip)
    torch.cuda.synchronize()
    assert int((tiled[..., 1] == n).sum()) > 0
    got = _captured(sen, big, scans, poses, trunc, clip)
    assert torch.equal(got.view(torch.int32), tiled.view(torch.int32))
    got = _captured(sen, small, scans, poses, trunc, clip)
    assert torch.equal(got.view(torch.int32), tiled[:12].contiguous().view(torch.int32))
