"""SDF fusion calls of more scans than one launch takes (32): a short last
launch, tile maxima made anew for each launch, blocks of the sparse volume
activated in a later launch than their call's first.

Dense: against the FP64 oracle as the other tests of the fusion, and to the
last bit against the same scans in calls of one launch each and against the
call without tile maxima (under stream capture).  Sparse: activation against
the oracle's, and to the last bit against calls of one launch each."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import sdf_ambiguous, to_dev
from test_gpu_sdf import SENSORS, compare, grid_points, run_gpu, sequence
from test_gpu_sdf_hash import EPS, ORIGIN, _export, _integrate, _key_map

pytestmark = pytest.mark.gpu

PER_LAUNCH = 32


@pytest.fixture(scope="module")
def rir():
    import torch
    import paper_2112_02779_amd as rir
    assert torch.cuda.is_available()
    return rir


@pytest.mark.parametrize("name", list(SENSORS))
@pytest.mark.parametrize("trunc,r_clip", [(0.5, 30.0), (0.0, 0.0)])
def test_two_launches_match_oracle(rir, name, trunc, r_clip):
    sm = SENSORS[name]()
    ranges, poses, seq = sequence(sm, PER_LAUNCH + 8)
    c = seq["poses"][0][:3, 3]
    vol = rir.Volume((4, 4, 2), (c[0] - 6.0, c[1] - 8.0, -1.0), 0.25)
    vox = run_gpu(rir, sm, vol, ranges, poses, trunc, r_clip)
    g = vol.to_grid(vox).cpu().numpy().reshape(-1, 2).astype(np.float64)
    pts = grid_points(vol)
    s_ref, w_ref = oracle.sdf_fuse(sm, ranges, poses, pts, trunc, r_clip)
    amb = sdf_ambiguous(sm, ranges, poses, pts, trunc, r_clip)
    R = (r_clip + trunc) if r_clip > 0 else float(ranges.max())
    compare(g[:, 0], g[:, 1], s_ref, w_ref, amb, 5e-7 * R + 1e-6, len(ranges))
    assert w_ref.max() == len(ranges)


@pytest.mark.parametrize("name", list(SENSORS))
@pytest.mark.parametrize("n", [33, 35, 40, 70])
def test_launches_of_a_call_equal_calls_of_one_launch(rir, name, n):
    """572 blocks: the last launch has fewer than 2048 block-scans (no tile
    maxima) with 33, 35 scans, more with 40 and 70 (three launches)."""
    import torch
    sm = SENSORS[name]()
    ranges, poses, seq = sequence(sm, n, seed=6)
    c = seq["poses"][n // 2][:3, 3]
    vol = rir.Volume((13, 11, 4), (c[0] - 10.4, c[1] - 8.8, -1.0), 0.1)
    one = run_gpu(rir, sm, vol, ranges, poses, 0.3, 25.0)
    parts = None
    for k in range(0, n, PER_LAUNCH):
        parts = run_gpu(rir, sm, vol, ranges[k:k + PER_LAUNCH], poses[k:k + PER_LAUNCH], 0.3, 25.0, voxels=parts)
    odd = run_gpu(rir, sm, vol, ranges[:21], poses[:21], 0.3, 25.0)
    odd = run_gpu(rir, sm, vol, ranges[21:], poses[21:], 0.3, 25.0, voxels=odd)
    plain, sen, dev = vol.alloc(), rir.Sensor.from_model(sm), to_dev(ranges)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rir.sdf_integrate(sen, vol, plain, dev, poses, 0.3, 25.0)
    graph.replay()
    torch.cuda.synchronize()
    assert float(one[..., 1].max()) > PER_LAUNCH  # some voxel is updated in more than one launch
    for other in (parts, odd, plain):
        assert torch.equal(one.view(torch.int32), other.view(torch.int32))


@pytest.mark.parametrize("name", list(SENSORS))
def test_sparse_launches(rir, name):
    n = 2 * PER_LAUNCH + 6
    sm = SENSORS[name]()
    ranges, poses, _ = sequence(sm, n, seed=11)
    one = _integrate(rir, sm, ranges, poses, 0.3, 30.0, 0.3, origin=ORIGIN)
    parts = None
    for k in range(0, n, PER_LAUNCH):
        parts = _integrate(rir, sm, ranges[k:k + PER_LAUNCH], poses[k:k + PER_LAUNCH], 0.3, 30.0, 0.3, vol=parts,
                           origin=ORIGIN)
    each = None
    for k in range(n):
        each = _integrate(rir, sm, ranges[k:k + 1], poses[k:k + 1], 0.3, 30.0, 0.3, vol=each, origin=ORIGIN)
    out = []
    for v in (one, parts, each):
        assert v.size()[1] == n
        b, vox = _export(v)
        order = np.lexsort(b[:, :3].T[::-1])
        out.append((b[order], vox[order].view(np.uint32)))
    for b, vox in out[1:]:
        np.testing.assert_array_equal(b, out[0][0])
        assert np.array_equal(vox, out[0][1])
    got = _key_map(out[0][0])
    inner = _key_map(oracle.sdf_activate(sm, ranges, poses, 0.3 - EPS, 30.0, 0.1, ORIGIN))
    outer = _key_map(oracle.sdf_activate(sm, ranges, poses, 0.3 + EPS, 30.0, 0.1, ORIGIN))
    assert set(inner) <= set(got) <= set(outer)
    for k, f in got.items():
        assert outer[k] <= f <= inner.get(k, 1 << 30), (k, f)
    # blocks first activated in the second and third launch
    first = np.array(list(got.values()))
    assert ((first >= PER_LAUNCH) & (first < 2 * PER_LAUNCH)).sum() > 20 and (first >= 2 * PER_LAUNCH).sum() > 5
