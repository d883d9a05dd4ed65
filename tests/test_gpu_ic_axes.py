"""The z pass that forms the initial displacement along all three axes, and its adjoint, at each
transform length.  The state against the FP64 oracle at 16^3 and 128^3 (32^3 and 64^3 elsewhere),
to the tolerance used there; the gradient along the noise field itself at 16^3, 64^3 and 256^3
against a central difference of step 1 +- 0.02: L = mean rho^2 - 1 is of second order in the
fluctuations, so the difference is exact but for their higher orders (a few times 0.02^2 of it) and
the rounding of the densities (1e-7 of 1 against a difference of 0.08 (L - 1) > 1e-4): 5e-3."""

import numpy as np
import pytest
import torch

import synth_inputs as si
from gpu_helpers import gpu_config, gpu_params, rel_l2, to_gpu, to_np
from oracle import sim as osim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lpt", [(16, 1), (16, 2), (128, 1)])
def test_initial_state_matches_oracle(n, lpt):
    import paper_2502_02294_amd as dhp
    print(f"initial conditions: n {n}, lpt {lpt}", flush=True)
    ocfg = osim.default_config(n=n, box=0.3 * n, lpt=lpt)
    s = dhp.Sim(gpu_config(ocfg), gpu_params(osim.Params()))
    w = si.white_noise(n, seed=3)
    s.init_from_noise(to_gpu(w))
    st = osim.initial_state(torch.from_numpy(w).double(), ocfg)
    for f in ("mom", "phi"):
        assert rel_l2(to_np(s.get(f)), getattr(st, {"mom": "p", "phi": "phi"}[f]).numpy()) < 1e-5, f
    s.close()


@pytest.mark.parametrize("n", [16, 64, 256])
def test_gradient_along_the_noise(n):
    import paper_2502_02294_amd as dhp
    print(f"gradient along the noise: n {n}", flush=True)
    a = 0.0105
    s = dhp.Sim(dhp.default_config(n=n, box=0.3 * n, a_init=0.01, subgrid=0))
    w = torch.from_numpy(np.asarray(si.white_noise(n, seed=4))).float().cuda()

    def density(x):
        s.forward(x.contiguous(), a)
        return s.get("q")[0].reshape(n, n, n)

    def loss(x):
        return float((density(x).double() / mean).square().mean() - 1.0)

    mean = float(density(w).double().mean())
    fd = (loss(1.02 * w) - loss(0.98 * w)) / 0.04
    g, _ = s.backward((2.0 / (n ** 3 * mean * mean) * density(w)).contiguous())
    dot = float((g.double().reshape(-1) * w.double().reshape(-1)).sum())
    assert abs(dot - fd) <= 5e-3 * abs(fd), (dot, fd)
    s.close()
