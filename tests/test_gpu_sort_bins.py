"""The particle sort at the edges of its cases: bins of 0, 1, 8, 9, 64, 65, 256, 257 and several
thousand particles (a lane, a wave, a workgroup; in LDS and, above 16384, in memory), and runs
of 64 bins that fit into a wave's LDS together or in parts.  The deposit over the sorted bins is
compared with a float64 CIC sum of the same float32 positions: a cell sums at most N / 64 + 70
rounded terms in a row, so 1e-5 relative up to 5000 particles a bin and 4e-5 for 20000."""

import numpy as np
import pytest
import torch

from gpu_helpers import to_gpu

pytestmark = pytest.mark.gpu


def _cic(pos, n):
    s = pos.astype(np.float64) - 0.5
    i = np.floor(s)
    w = s - i
    i = i.astype(np.int64)
    out = np.zeros(n ** 3)
    for o in range(8):
        b = (o & 1, o >> 1 & 1, o >> 2)
        j = [(i[d] + b[d]) % n for d in range(3)]
        wt = np.ones(pos.shape[1])
        for d in range(3):
            wt = wt * (w[d] if b[d] else 1.0 - w[d])
        np.add.at(out, (j[2] * n + j[1]) * n + j[0], wt)
    return out


def _fill(n, sizes, seed):
    """n^3 particles in random order: bins of the given sizes, the rest one per bin."""
    r = np.random.default_rng(seed)
    total = n ** 3
    bins = r.permutation(total)
    base, used = [], 0
    for k, b in zip(sizes, bins):
        if used + k > total:
            break
        base.append(np.full(k, b))
        used += k
    base.append(bins[len(sizes):len(sizes) + total - used])
    base = np.concatenate(base)
    base = r.permutation(np.concatenate([base, base[: total - base.size]]))
    cell = np.stack([base % n, base // n % n, base // (n * n)])
    pos = (cell + 0.5 + r.uniform(0.01, 0.99, cell.shape)).astype(np.float32)
    return np.where(pos >= n, pos - n, pos).astype(np.float32)


CASES = {
    "lane": ([8, 9, 7, 2] * 40, 1e-5),
    "edge": ([128, 129, 127, 8, 130] * 6, 1e-5),
    "wave": ([64, 65, 256, 255, 63, 9] * 6, 1e-5),
    "neighbours": ([200] * 120, 1e-5),
    "workgroup": ([257, 300, 5000, 256], 1e-5),
    "memory": ([20000, 257, 12], 4e-5),
}


@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("kind", sorted(CASES))
def test_deposit_over_bins_of_every_size(n, kind):
    import paper_2502_02294_amd as dhp
    sizes, tol = CASES[kind]
    print(f"sort bins: n {n}, {kind}", flush=True)
    pos = _fill(n, sizes, seed=n)
    s = dhp.Sim(dhp.default_config(n=n))
    zero = torch.zeros(n, n, n, dtype=torch.float32, device="cuda")
    ref = _cic(pos, n)
    m_dm = 1.0 - 0.05 / 0.3
    for _ in range(2):   # the second finds the workspace as the first left it
        d = s.stage_deposit(zero, to_gpu(pos)).double().cpu().numpy().reshape(-1)
        # delta = m_dm CIC - 1, whose own rounding is one of a number of order 1
        assert np.all(np.abs(d - (m_dm * ref - 1.0)) <= tol * m_dm * ref + 2e-7)
    s.close()
