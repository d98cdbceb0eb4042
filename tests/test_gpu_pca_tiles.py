"""PCA normals where their tiles and their range test can go wrong: images
smaller than a tile of 32 x 8 pixels, remainders of one column or row, windows
that wrap more than the image is wide, and ranges on the limit of the window's
range test or one float away from it (FP32 cannot decide those).  Against the
FP64 oracle; the output's FP32 rounding bounds the angle (2e-7 rad), for
normals whose two smallest eigenvalues are apart."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [1, 2, 3])
@pytest.mark.parametrize("H,W", [(2, 4), (7, 31), (8, 32), (9, 33), (17, 100)])
def test_pca_tile_edges_and_limit_ranges(H, W, half):
    import paper_2112_02779_amd as rir
    sm = synth.staggered_sensor(H, W, r0=0.015) if W == 100 else synth.uniform_sensor(H, W)
    rng = np.random.default_rng(100 * H + half)
    # |r - rc| = edge_rel rc exactly for (8, 9), (8, 7) and (16, 18), and the
    # floats next to those
    base = np.array([8.0, 9.0, 7.0, 16.0, 18.0, 14.0], np.float32)
    pool = np.concatenate([base, np.nextafter(base, np.float32(0)), np.nextafter(base, np.float32(99)), [0.0]])
    imgs = rng.choice(pool.astype(np.float32), size=(2, H, W))
    imgs[1] = np.where(rng.random((H, W)) < 0.8, rng.choice(pool[[0, 1, 6, 7, 12, 13]], size=(H, W)), imgs[1])
    n, valid = rir.normals_pca(rir.Sensor.from_model(sm), to_dev(imgs), half=half, edge_rel=0.125)
    n = n.cpu().numpy().astype(np.float64)
    valid = valid.cpu().numpy().astype(bool)
    for k in range(2):
        n_ref, v_ref, lam = oracle.normals_pca(sm, imgs[k], half=half, edge_rel=0.125)
        top = lam[..., 2]
        clear = ~((top > 0) & (np.abs(lam[..., 1] - 1e-6 * top) <= 1e-9 * top))
        np.testing.assert_array_equal(valid[k][clear], v_ref[clear])
        assert np.all(n[k][~valid[k]] == 0)
        both = valid[k] & v_ref & (lam[..., 1] - lam[..., 0] > 1e-6 * top)
        c = np.linalg.norm(np.cross(n[k][both], n_ref[both]), axis=-1)
        d = np.sum(n[k][both] * n_ref[both], axis=-1)
        assert np.max(np.arctan2(c, d), initial=0.0) < 2e-7


@pytest.mark.parametrize("prec", [0, 1])
def test_pca_records_of_mixed_sizes(prec):
    """Records tiles of two image sizes in one batch (64 x 1000: a remainder
    of 8 columns): every pair as in a batch of its own, to the last bit."""
    import paper_2112_02779_amd as rir
    prm = rir.make_params(levels=3, iters=[4, 4, 4], delta=0.5, normal_window=1, precision=prec)
    ctx = rir.Context(0)
    pairs = []
    for k, sm in enumerate([synth.uniform_sensor(64, 1024), synth.staggered_sensor(32, 500, r0=0.015),
                            synth.staggered_sensor(64, 1000, r0=0.015)]):
        p = synth.gen_pair(synth.CONFIGS["pair64"], 60 + k, sensor=sm)
        pairs.append((rir.Sensor.from_model(sm), to_dev(p.src), to_dev(p.dst)))
    T, _ = rir.icp_batch(ctx, prm, pairs)
    T = T.cpu().numpy()
    for k, p in enumerate(pairs):
        one, _ = rir.icp_batch(ctx, prm, [p])
        np.testing.assert_array_equal(T[k], one.cpu().numpy()[0])
