"""Every sample of a batch takes part in the training gradient, at the batch
sizes where its split changes: only one sample has features, so the whole
gradient of the first layer's weights is its own.  Against the FP64 oracle;
tolerance as in the other test of those sizes (two bf16 factors, each off by
2^-8 at most: 2^-7 of the block's largest entry)."""
import numpy as np
import pytest

import oracle
from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,at", [(1, 0), (17, 16), (65, 64), (8192, 8191), (8193, 8192), (8193, 8191), (16384, 16383),
                                  (16385, 16384), (32769, 32768), (131073, 131072), (131073, 131071), (200000, 0)])
def test_one_samples_gradient(B, at):
    import torch
    import paper_2112_02779_amd as rir
    P = rir.init_mlp_params(5)
    P[896:960] = np.random.default_rng(1).normal(size=64) * 0.1
    P = rir.join_params(*rir.split_params(P))
    rng = np.random.default_rng(B + at)
    f = np.zeros((B, 14), np.float32)
    f[at] = rng.normal(size=14) * 2.0
    y = (rng.random(B) < 0.7).astype(np.float32)
    _, g = rir.Mlp(P).train_step(to_dev(f), to_dev(y), lr=0.0, want_grads=True)
    torch.cuda.synchronize()
    _, go = oracle.mlp_loss_grad(P, f, y)
    g, go = g.cpu().numpy().astype(np.float64)[:896], np.asarray(go)[:896]
    assert np.abs(go).max() > 0.01 / B
    assert np.abs(g - go).max() <= 2.0 ** -7 * np.abs(go).max()
