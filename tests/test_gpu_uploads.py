"""The per-step tables reach the device as launch arguments (one sample, a few samples) or, for
larger batches, through pinned memory: a sample of a batch of any size takes the same steps as
the sample alone, bit for bit, and its loss and CFL schedule, handed back through host memory,
are the same."""

import numpy as np
import pytest
import torch

import synth_inputs as si
from gpu_helpers import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("samples", [2, 13, 14, 15, 16, 40])
def test_batches_of_every_upload_size(samples):
    import paper_2502_02294_amd as dhp
    n = 16
    print(f"uploads: {samples} samples", flush=True)
    white = to_gpu(np.stack([si.white_noise(n, 60 + i) for i in range(samples)]))
    target = torch.full_like(white, 0.4)
    kw = dict(n=n, box=2.5, subgrid=2)
    b = dhp.Sim(dhp.default_config(batch=samples, **kw))
    b.forward(white, 0.012)
    loss = b.loss(target)
    last = samples - 1
    s = dhp.Sim(dhp.default_config(sf_seed=102 + last, **kw))
    s.forward(white[last].contiguous(), 0.012)
    assert s.get_schedule() == b.get_sample_schedule(last)
    assert torch.equal(s.get("q"), b.get("q")[last])
    assert torch.equal(s.get("mom"), b.get("mom")[last])
    assert s.loss(target[last].contiguous()) == loss[last]
    s.close()
    b.close()
