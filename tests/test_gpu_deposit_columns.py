"""The column walk of the CIC deposits where its cases meet: bins of 0, 1, 2 (loaded ahead), 3,
16 (a thread's own loop), 17, 64 and 65 particles (a wave's), on both sides of the seams between
columns, walks and the periodic boundary, for walks of one plane (16^3 to 64^3) and of four
(128^3), and over a batch against single runs.  Against a float64 CIC sum of the same float32
positions: a bin's sum rounds at most 70 + 20 times, a cell's 8 more and a weight 4 times, so
100 x 2^-23 = 1.2e-5 relative, and the rounding of delta + 1, a number of order 1 (2e-7)."""

import numpy as np
import pytest
import torch

import synth_inputs as si
from gpu_helpers import to_gpu
from test_gpu_sort_bins import _cic

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 2, 3, 16, 17, 64, 65]


def _seams(n, seed, runs):
    """n^3 particles: bins of the sizes above at the seams (and their neighbours), the rest of
    the particles anywhere; in random order or (runs) a bin's particles one after the other."""
    r = np.random.default_rng(seed)
    edge = np.array([0, 1, 3, 4, 15, n - 1])
    cells = np.stack(np.meshgrid(edge, edge, edge, indexing="ij")).reshape(3, -1)
    cells = cells[:, r.permutation(cells.shape[1])][:, : max(8, n ** 3 // 64)]
    k = np.array(SIZES)[np.arange(cells.shape[1]) % len(SIZES)]
    cell = np.repeat(cells, k, axis=1)
    rest = n ** 3 - cell.shape[1]
    cell = np.concatenate([cell, r.integers(0, n, (3, rest))], axis=1)
    pos = (cell + 0.5 + r.uniform(0.0, 0.999, cell.shape)).astype(np.float32)
    pos = np.where(pos >= n, pos - n, pos).astype(np.float32)
    return pos if runs else pos[:, r.permutation(n ** 3)]


@pytest.mark.parametrize("n,runs", [(16, False), (32, False), (32, True), (64, False), (128, False),
                                    (128, True)])
def test_deposit_at_the_seams(n, runs):
    import paper_2502_02294_amd as dhp
    print(f"deposit seams: n {n}, runs {runs}", flush=True)
    s = dhp.Sim(dhp.default_config(n=n))
    pos = _seams(n, 7 * n, runs)
    zero = torch.zeros(n, n, n, dtype=torch.float32, device="cuda")
    d = s.stage_deposit(zero, to_gpu(pos)).double().cpu().numpy().reshape(-1)
    ref = (1.0 - 0.05 / 0.3) * _cic(pos, n)
    assert np.all(np.abs(d - (ref - 1.0)) <= 1.2e-5 * ref + 2e-7)
    s.close()


def test_batched_walks_match_single_runs():
    # 32 samples of 32^3 walk two planes where one sample walks one: the same sums, bit for bit
    import paper_2502_02294_amd as dhp
    n, S, i = 32, 32, 31
    print(f"deposit walks: n {n}, batch {S}", flush=True)
    white = np.stack([si.white_noise(n, seed=60 + k) for k in range(S)])
    kw = dict(n=n, box=10.0, subgrid=0)
    b = dhp.Sim(dhp.default_config(batch=S, **kw))
    s = dhp.Sim(dhp.default_config(**kw))
    b.init_from_noise(to_gpu(white))
    s.init_from_noise(to_gpu(white[i]))
    b.run_steps(2)
    s.run_steps(2)
    for f in ("q", "pos", "mom", "phi"):
        assert torch.equal(b.get(f)[i], s.get(f)), f
    b.close()
    s.close()
