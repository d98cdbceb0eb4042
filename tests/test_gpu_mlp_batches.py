"""The training gradient at the batch sizes where its split changes: partial
16-sample tiles, the last batch of 16, 32 and 64 samples a wavefront, and the
first beyond it.

Tolerance: an activation or delta within FP32 rounding of a bf16 tie may be
rounded the other way than in the FP64 oracle, which moves a sample's term by
up to 2^-8 of itself in each of its two factors; the FP32 sums are far below
that.  So 2^-7 of a block's largest entry."""
import numpy as np
import pytest

import oracle
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 65, 8192, 8193, 16384, 16385, 32769])
def test_gradient_at_split_edges(B):
    import torch
    import paper_2112_02779_amd as rir
    P = rir.init_mlp_params(5)
    P[896:960] = np.random.default_rng(1).normal(size=64) * 0.1
    P[5056:5120] = np.random.default_rng(2).normal(size=64) * 0.1
    P = rir.join_params(*rir.split_params(P))
    rng = np.random.default_rng(B)
    f = rng.normal(size=(B, 14)).astype(np.float32)
    y = (rng.random(B) < 0.7).astype(np.float32)
    net = rir.Mlp(P)
    loss, g = net.train_step(to_dev(f), to_dev(y), lr=0.0, want_grads=True)
    torch.cuda.synchronize()
    lo, go = oracle.mlp_loss_grad(P, f, y)
    g = g.cpu().numpy().astype(np.float64)
    assert abs(float(loss.cpu()) - lo) < 1e-5 * max(1.0, abs(lo))
    for a, b in ((0, 896), (896, 960), (960, 5056), (5056, 5120), (5120, 5184), (5184, 5185)):
        assert np.abs(g[a:b] - go[a:b]).max() <= 2.0 ** -7 * np.abs(go[a:b]).max() + 1e-9, (a, b)
