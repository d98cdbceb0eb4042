"""A training step captured into a graph after a larger batch ran: the records
that the larger batch allocated must hold those of every smaller one, since
nothing can be allocated while a stream is captured.  (The split of a batch
takes 16, 32 or 64 samples a wavefront, so a smaller batch can have more
records: 512 at 8192 samples, 316 at 20000.)"""
import numpy as np
import pytest

from parity_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("large,small", [(20000, 8192), (8193, 8192), (16385, 16384), (8192, 17)])
def test_smaller_batch_captured_after_a_larger_one(large, small):
    import torch
    import paper_2112_02779_amd as rir
    rng = np.random.default_rng(large)
    f = to_dev(rng.normal(size=(large, 14)).astype(np.float32))
    y = to_dev((rng.random(large) < 0.7).astype(np.float32))
    P = rir.init_mlp_params(5)
    net, ref = rir.Mlp(P), rir.Mlp(P)
    net.train_step(f, y, lr=0.0)
    torch.cuda.synchronize()
    fs, ys = f[:small].contiguous(), y[:small].contiguous()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        loss, grads = net.train_step(fs, ys, lr=0.0, want_grads=True)
    lo, go = ref.train_step(fs, ys, lr=0.0, want_grads=True)
    for _ in range(3):
        loss.zero_()
        grads.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(loss, lo) and torch.equal(grads, go)
