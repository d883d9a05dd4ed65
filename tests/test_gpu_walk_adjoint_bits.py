"""A sample's gradient is the same bits alone and in a batch.  The number of samples sets how
many segments the y and z walks cut a pencil into (below: 8 cells a segment for one sample, 16
or 32 for the batch), so the walks' adjoint must not depend on the cut."""

import numpy as np
import pytest
import torch

import synth_inputs as si
from gpu_helpers import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,samples,dual,steps", [(32, 70, 0, 2), (64, 9, 0, 3), (64, 9, 1, 2),
                                                  (64, 32, 0, 2), (128, 2, 0, 2)])
def test_gradient_is_the_same_alone_and_in_a_batch(n, samples, dual, steps):
    import paper_2502_02294_amd as dhp
    print(f"walk adjoint: n {n}, {samples} samples, dual {dual}", flush=True)
    kw = dict(n=n, box=n * 10.0 / 64, subgrid=2, dual_energy=dual)
    white = to_gpu(np.stack([si.white_noise(n, 60 + i % 5) for i in range(samples)]))
    target = torch.full_like(white, 0.4)

    def gradient(w, t, seed, batch):
        s = dhp.Sim(dhp.default_config(sf_seed=seed, batch=batch, **kw))
        s.init_from_noise(w)
        s.run_steps(steps)
        if batch == 1:
            s.set_schedule(s.get_schedule())
        else:
            for i in range(batch):
                s.set_sample_schedule(i, s.get_sample_schedule(i))
        s.forward(w, 1.0)
        s.loss(t)
        g = s.backward()[0].clone()
        s.close()
        return g

    together = gradient(white, target, 102, samples)
    for i in (0, samples - 1):
        alone = gradient(white[i].contiguous(), target[i].contiguous(), 102 + i, 1)
        assert torch.equal(alone, together[i]), (i, (alone - together[i]).abs().max())
