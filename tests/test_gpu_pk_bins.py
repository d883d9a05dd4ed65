"""The power spectrum's binning over its splits: 1 to n/2 bins (a thread per bin and share of the
modes, bins padded to a power of two), boxes with two and with eight modes a thread and a last
block that is not full.  Against the FP64 oracle on white density fields, whose modes are all of
the transform's rounding (about 2e-7 log2 n^3 < 5e-6 of a mode, its square twice that): 1e-5."""

import numpy as np
import pytest
import torch

from gpu_helpers import gpu_config, gpu_params, to_gpu
from oracle import observe, sim as osim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nbins", [(16, 1), (16, 8), (64, 20), (64, 32), (128, 3), (128, 64)])
def test_power_spectrum_bins(n, nbins):
    import paper_2502_02294_amd as dhp
    print(f"power spectrum: n {n}, {nbins} bins", flush=True)
    ocfg = osim.default_config(n=n, box=0.25 * n)
    s = dhp.Sim(gpu_config(ocfg), gpu_params(osim.Params()))
    rho = np.random.default_rng(n + nbins).uniform(0.5, 1.5, (n, n, n)).astype(np.float32)
    q = np.zeros((5, n, n, n), dtype=np.float32)
    q[0] = rho
    q[4] = 1.0
    s.set("q", to_gpu(q))
    pk, _, _ = s.power_spectrum(nbins)
    ref = observe.power_spectrum(torch.from_numpy(rho.astype(np.float64)), ocfg.f_b, ocfg.box,
                                 nbins)[0].numpy()
    assert np.all(np.abs(np.asarray(pk) - ref) <= 1e-5 * ref)
    s.close()
