"""SDF fusion with layers dropped by the scans' tile maxima, against the same
call without them (under stream capture no tile maxima are used): the volumes
must be equal to the last bit, whatever the sensor, the poses, the truncation
and the holes of the scans."""
import numpy as np
import pytest
import torch

import synth
import paper_2112_02779_amd as rir

pytestmark = pytest.mark.gpu

# at least 2048 block-scans, from which on the tile maxima are used
NB, SCANS, VOXEL = (13, 11, 4), 5, 0.11


def _scans(sm, rng, holes):
    """Rough range images: sectors of constant range with noise, holes, far and invalid values."""
    H, W = sm.H, sm.W
    r = np.repeat(rng.uniform(0.3, 25.0, size=(SCANS, H, -(-W // 7))), 7, axis=2)[:, :, :W]
    r = r + rng.normal(0, 0.05, size=r.shape)
    r[rng.random(r.shape) < holes] = 0.0
    bad = rng.random(r.shape)
    r[bad < 0.01] = np.nan
    r[bad > 0.99] = np.inf
    r[(bad > 0.5) & (bad < 0.51)] = -1.0
    return torch.from_numpy(r.astype(np.float32)).to("cuda:0")


def _poses(rng, kind):
    T = np.zeros((SCANS, 4, 4))
    for k in range(SCANS):
        ang = rng.uniform(0, 2 * np.pi) if kind == "level" else rng.uniform(0, np.pi)
        axis = np.array([0.0, 0.0, 1.0]) if kind == "level" else synth.unit_vector(rng)
        P = synth.make_pose(synth.rot_axis_angle(axis, ang), rng.uniform([-14, -14, -3], [14, 14, 6]))
        T[k] = synth.inv_pose(P)
        if kind == "affine":  # accepted as any finite matrix is
            T[k, :3, :3] = T[k, :3, :3] @ np.diag(rng.uniform(0.5, 1.5, size=3))
    return T


@pytest.mark.parametrize("shape,sensor", [((32, 256), "uniform"), ((64, 1000), "uniform"), ((48, 333), "staggered"),
                                          ((3, 64), "uniform"), ((2, 17), "staggered"), ((16, 40), "wide")])
@pytest.mark.parametrize("poses", ["level", "tilted", "affine"])
@pytest.mark.parametrize("trunc,clip", [(0.3, 12.0), (0.0, 0.0), (0.25, 0.0)])
def test_tile_maxima_change_nothing(shape, sensor, poses, trunc, clip):
    rng = np.random.default_rng(hash((shape, len(sensor), len(poses))) % 1000)
    sm = synth.staggered_sensor(*shape, r0=0.05) if sensor == "staggered" else synth.uniform_sensor(*shape)
    if sensor == "wide":  # azimuth offsets of up to 3 rad and nearly the whole sphere in view
        sm = synth.uniform_sensor(*shape, fov_up_deg=85.0, fov_down_deg=-85.0)
        sm.theta = rng.uniform(-3.0, 3.0, size=sm.H)
    sen = rir.Sensor.from_model(sm)
    vol = rir.Volume(NB, tuple(-8.0 * VOXEL * np.array(NB)), VOXEL)
    for holes in (0.05, 0.97):
        scans, T = _scans(sm, rng, holes), _poses(rng, poses)
        with_tiles, without = vol.alloc(), vol.alloc()
        rir.sdf_integrate(sen, vol, with_tiles, scans, T, trunc, clip)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            rir.sdf_integrate(sen, vol, without, scans, T, trunc, clip)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(with_tiles.view(torch.int32), without.view(torch.int32))
        if holes < 0.5:
            assert int((with_tiles[..., 1] > 0).sum()) > 0


def test_tile_slots_of_several_streams():
    """More streams than slots on one sensor: every call gives the same volume."""
    rng = np.random.default_rng(3)
    sm = synth.uniform_sensor(32, 512)
    sen = rir.Sensor.from_model(sm)
    vol = rir.Volume(NB, tuple(-8.0 * VOXEL * np.array(NB)), VOXEL)
    scans, T = _scans(sm, rng, 0.05), _poses(rng, "level")
    want = vol.alloc()
    rir.sdf_integrate(sen, vol, want, scans, T, 0.3, 12.0)
    got = [vol.alloc() for _ in range(8)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(8)]
    for k, st in enumerate(streams):
        rir.sdf_integrate(sen, vol, got[k], scans, T, 0.3, 12.0, stream=st)
    torch.cuda.synchronize()
    for g in got:
        assert torch.equal(g.view(torch.int32), want.view(torch.int32))
