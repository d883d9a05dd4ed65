"""The training step's packing and splits.  Adam writes the packed (matrix-core) weights along with
the weights: after training they have to be those that loading the weights packs, so that the
network and its input gradient agree bit for bit, at every parameter.  The gradient takes the batch
in groups of 32 samples, two waves of 16 each and two groups a block: counts on both sides of each,
against the oracle with the tolerance of the larger batches."""

import numpy as np
import pytest
import torch

from gpu_helpers import rel_l2, to_gpu
from oracle import mlp as omlp
from test_gpu_mlp import BWD_TOL, _inputs, _theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [17, 512])
def test_training_keeps_the_packed_weights(batch):
    import paper_2502_02294_amd as dhp
    print(f"packed weights after training: batch {batch}", flush=True)
    net, fresh = dhp.Mlp(seed=3), dhp.Mlp()
    x, y = net.sample(2048, seed=9)
    net.train(x, y, steps=5, batch=batch, lr=3e-3)
    fresh.set_weights(net.weights())
    z = to_gpu(_inputs(400, seed=21))
    gout = to_gpu(np.random.default_rng(22).normal(size=(2, 400)).astype(np.float32))
    assert torch.equal(net.eval(z), fresh.eval(z))
    assert torch.equal(net.vjp(z, gout), fresh.vjp(z, gout))


@pytest.mark.parametrize("count", [1, 16, 17, 32, 33, 64, 65])
def test_gradient_of_small_batches(count):
    import paper_2502_02294_amd as dhp
    print(f"weight gradient: {count} samples", flush=True)
    net = dhp.Mlp(seed=6)
    x = _inputs(count, seed=13)
    y = np.random.default_rng(14).normal(0.0, 3.0, (2, count)).astype(np.float32)
    loss, g = net.grad(to_gpu(x), to_gpu(y))
    th = _theta(net).requires_grad_(True)
    L = omlp.loss(th, torch.from_numpy(x).double(), torch.from_numpy(y).double(), bf16=True)
    ref, = torch.autograd.grad(L, th)
    assert abs(loss - float(L.detach())) < 1e-4 * float(L.detach())
    assert rel_l2(g, ref.numpy()) < BWD_TOL
