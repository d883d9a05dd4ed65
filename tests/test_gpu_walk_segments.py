"""The y and z sweeps cut a pencil into segments by how many waves the launch has: one sample
and the same sample in a batch take different segment lengths.  The forward is the same bit
for bit; the adjoint rounds its first output of a segment differently (one float32 rounding,
6e-8, in one cell of eight), so gradients over two steps agree to 1e-5."""

import pytest
import torch

import synth_inputs as si
from gpu_helpers import rel_l2, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,samples,dual", [(16, 5, 0), (64, 9, 0), (64, 9, 1), (128, 2, 0)])
def test_segment_length_does_not_change_results(n, samples, dual):
    import numpy as np
    import paper_2502_02294_amd as dhp
    print(f"walk segments: n {n}, {samples} samples, dual {dual}", flush=True)
    kw = dict(n=n, box=n * 10.0 / 64, subgrid=2, dual_energy=dual)
    white = to_gpu(np.stack([si.white_noise(n, 40 + i) for i in range(samples)]))
    target = torch.full_like(white, 0.4)
    b = dhp.Sim(dhp.default_config(batch=samples, **kw))
    b.init_from_noise(white)
    b.run_steps(2)
    q = b.get("q")
    sched = [b.get_sample_schedule(i) for i in range(samples)]
    for i in range(samples):
        b.set_sample_schedule(i, sched[i])
    b.forward(white, 1.0)
    b.loss(target)
    grad, _ = b.backward()
    b.close()
    last = samples - 1
    s = dhp.Sim(dhp.default_config(sf_seed=102 + last, **kw))
    s.init_from_noise(white[last].contiguous())
    s.run_steps(2)
    assert torch.equal(s.get("q"), q[last])
    s.set_schedule(sched[last])
    s.forward(white[last].contiguous(), 1.0)
    s.loss(target[last].contiguous())
    one, _ = s.backward()
    assert rel_l2(to_np(one), to_np(grad[last])) < 1e-5
    s.close()
