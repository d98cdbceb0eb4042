"""SDF fusion with layers dropped by the scans' tile maxima where a layer lies
exactly around the sensor's axis or beside it: voxel sizes of one mantissa bit,
rotations without a rounding error, the sensor over a block's centre, a voxel
column, a block's face or its corner.  Against the same scans without tile
maxima (a dense call under stream capture; a sparse volume of fewer than 2048
blocks fused scan by scan): equal to the last bit."""
import numpy as np
import pytest
import torch

import synth
import paper_2112_02779_amd as rir

pytestmark = pytest.mark.gpu

TURNS = {
    "identity": np.eye(3),
    "yaw90": np.array([[0.0, -1.0, 0.0], [1.0, 0.0, 0.0], [0.0, 0.0, 1.0]]),
    "on its side": np.array([[0.0, 0.0, 1.0], [0.0, 1.0, 0.0], [-1.0, 0.0, 0.0]]),
}
# the sensor's place in its block, in voxels
PLACES = {"centre": (7.5, 7.5, 7.5), "centre, between layers": (7.5, 7.5, 3.0), "column": (4.0, 11.0, 7.5),
          "face": (15.5, 7.5, 2.0), "corner": (15.5, 15.5, 15.5)}


def _scans(sm, n, blind):
    """Every row near 10 m; blind: the lowest beam sees nothing."""
    r = np.full((n, sm.H, sm.W), 10.0, np.float32)
    r += np.float32(0.25) * np.arange(n, dtype=np.float32)[:, None, None]
    if blind:
        r[:, -1] = 0.0
    return torch.from_numpy(r).to("cuda:0")


def _pose(turn):
    T = np.zeros((1, 4, 4))
    T[0, :3, :3] = TURNS[turn]
    T[0, 3, 3] = 1.0
    return T


@pytest.mark.parametrize("turn", list(TURNS))
@pytest.mark.parametrize("place", list(PLACES))
@pytest.mark.parametrize("voxel,fov,blind", [(0.25, 16.6, True), (0.25, 80.0, False), (0.5, 45.0, True),
                                             (0.125, 16.6, False)])
def test_dense_layers_around_the_axis(voxel, fov, blind, place, turn):
    sm = synth.uniform_sensor(32, 1024, fov_up_deg=fov, fov_down_deg=-fov)
    sen = rir.Sensor.from_model(sm)
    nb = (13, 13, 13)  # 2197 blocks: one scan is enough for the tile maxima
    vol = rir.Volume(nb, tuple(-voxel * (16.0 * 6 + p) for p in PLACES[place]), voxel)
    scan, T = _scans(sm, 1, blind), _pose(turn)
    tiled, plain = vol.alloc(), vol.alloc()
    rir.sdf_integrate(sen, vol, tiled, scan, T, 0.3, 30.0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rir.sdf_integrate(sen, vol, plain, scan, T, 0.3, 30.0)
    graph.replay()
    torch.cuda.synchronize()
    assert int((plain[6, 6, 6, ..., 1] > 0).sum()) > 0  # the sensor's own block
    assert torch.equal(tiled.view(torch.int32), plain.view(torch.int32))


@pytest.mark.parametrize("turn", list(TURNS))
@pytest.mark.parametrize("place", list(PLACES))
def test_sparse_layers_around_the_axis(place, turn):
    sm = synth.uniform_sensor(32, 1024)
    sen = rir.Sensor.from_model(sm)
    voxel, n = 0.25, 5
    scans, T = _scans(sm, n, True), np.repeat(_pose(turn), n, 0)
    origin = tuple(-voxel * p for p in PLACES[place])
    vols = [rir.BlockVolume(voxel, 4000, origin) for _ in range(2)]
    vols[0].integrate(sen, scans, T, 0.3, 30.0, 10.0)
    for k in range(n):
        vols[1].integrate(sen, scans[k:k + 1], T[k:k + 1], 0.3, 30.0, 10.0)
    size = vols[0].size()[0]
    assert size == vols[1].size()[0] < 2048 <= n * size
    out = []
    for v in vols:
        b, vox = v.export()
        b = b.cpu().numpy()
        order = np.lexsort(b[:, :3].T[::-1])
        out.append((b[order], vox.cpu().numpy()[order].view(np.uint32)))
    np.testing.assert_array_equal(out[0][0], out[1][0])
    own = int(np.flatnonzero((out[1][0][:, :3] == 0).all(1))[0])
    assert (out[1][1][own, ..., 1] != 0).sum() > 0
    assert np.array_equal(out[0][1], out[1][1])
