"""The reverse pass's vector deposit over bins of every size: it takes the particles' ids in bin
order beside their weights, and sums bins of more than 16 particles by whole waves.

As a stage, against a float64 CIC sum of the same float32 inputs, over the bins of the scalar
deposit's tests: a corner's sum rounds at most N / 64 + 70 + 20 times for bins of up to N
particles, a product 4 times and a cell's sum 8, relative to the sum of the absolute terms, so
200 x 2^-23 = 2.4e-5 up to 5000 particles a bin and 500 x 2^-23 = 6e-5 for 20000.

In the gradient of a run whose particles collapse (plane waves that focus on one point: bins of
up to several hundred particles), a sample of a batch against the sample alone, and steps whose
sort was taped, stored or made again, bit for bit."""

import numpy as np
import pytest
import torch

from gpu_helpers import to_gpu, to_np
from oracle import ics, sim as osim
from test_gpu_deposit_columns import _seams
from test_gpu_sort_bins import CASES, _fill

pytestmark = pytest.mark.gpu
torch.set_default_dtype(torch.float64)


def _cic_vec(pos, vec, n):
    """float64 CIC sums of vec and of |vec|, [3, n^3] each"""
    s = pos.astype(np.float64) - 0.5
    i = np.floor(s)
    w = s - i
    i = i.astype(np.int64)
    out, mag = np.zeros((3, n ** 3)), np.zeros((3, n ** 3))
    for o in range(8):
        b = (o & 1, o >> 1 & 1, o >> 2)
        j = [(i[d] + b[d]) % n for d in range(3)]
        c = (j[2] * n + j[1]) * n + j[0]
        wt = np.ones(pos.shape[1])
        for d in range(3):
            wt = wt * (w[d] if b[d] else 1.0 - w[d])
        for k in range(3):
            out[k] += np.bincount(c, wt * vec[k], n ** 3)
            mag[k] += np.bincount(c, wt * np.abs(vec[k]), n ** 3)
    return out, mag


def _compare(n, pos, tol):
    import paper_2502_02294_amd as dhp
    r = np.random.default_rng(n)
    vec = r.standard_normal(pos.shape).astype(np.float32)
    before = r.standard_normal((3, n, n, n)).astype(np.float32)
    ref, mag = _cic_vec(pos, vec, n)
    s = dhp.Sim(dhp.default_config(n=n))
    zero = torch.zeros(n, n, n, dtype=torch.float32, device="cuda")
    outs = []
    for _ in range(2):
        out = to_gpu(before)
        s.stage_deposit_vec(to_gpu(pos), to_gpu(vec), out)
        outs.append(out)
        s.stage_deposit(zero, to_gpu(pos))   # a sort that keeps no ids in between
    s.close()
    assert torch.equal(outs[0], outs[1])
    b = before.reshape(3, -1).astype(np.float64)
    got = to_np(outs[0]).reshape(3, -1)
    assert np.all(np.abs(got - (b + ref)) <= tol * mag + 1.2e-7 * np.abs(b + ref) + 1e-12)


@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("kind", sorted(CASES))
def test_bins_of_every_size(n, kind):
    print(f"vector deposit: n {n}, {kind}", flush=True)
    _compare(n, _fill(n, CASES[kind][0], seed=n), 6e-5 if kind == "memory" else 2.4e-5)


@pytest.mark.parametrize("n,runs", [(16, False), (32, True), (64, False), (128, False)])
def test_seams(n, runs):
    print(f"vector deposit seams: n {n}, runs {runs}", flush=True)
    _compare(n, _seams(n, 7 * n, runs), 2.4e-5)


N, STEPS, ALPHA = 16, 8, 0.7


def _focusing_noise(cfg, seed):
    """White noise whose displacement is -(ALPHA / k) sin k (x - n/2) along each axis, k the
    smallest wavenumber, and 1% of noise"""
    i, k = np.arange(N) + 0.5, 2 * np.pi / N
    c = np.cos(k * (i - N / 2))
    w = c[None, None, :] + c[None, :, None] + c[:, None, None]
    _, x, _ = ics.initial_state(torch.from_numpy(w).double(), cfg)
    d = ((x - ics.lattice(N).double() + N / 2) % N - N / 2)[0].reshape(N, N, N).numpy()
    w *= -ALPHA / k / (d[0, 0] @ np.sin(k * (i - N / 2)) / (N / 2))
    r = np.random.default_rng(seed)
    return (w + 0.01 * np.abs(w).max() * r.standard_normal(w.shape)).astype(np.float32)


def test_gradient_of_a_collapsing_run():
    import paper_2502_02294_amd as dhp
    print("vector deposit: collapsing run", flush=True)
    kw = dict(n=N, box=N * 10.0 / 64, a_init=0.05, dlna_max=0.15, subgrid=0)
    cfg = osim.default_config(**kw)
    white = np.stack([_focusing_noise(cfg, s) for s in (0, 1)])
    target = (0.2 + 0.7 * np.random.default_rng(4).random(white.shape)).astype(np.float32)
    st, sched = osim.run(osim.initial_state(torch.from_numpy(white[1]).double(), cfg), cfg,
                         osim.Params(), nsteps=STEPS)
    cell = np.floor(st.x.numpy() - 0.5).astype(np.int64) % N
    size = np.bincount((cell[2] * N + cell[1]) * N + cell[0], minlength=N ** 3)
    for lo, hi in ((1, 2), (3, 16), (17, 64), (129, N ** 3)):
        assert ((size >= lo) & (size <= hi)).any(), (lo, hi)

    def gradient(w, t, batch, limit):
        s = dhp.Sim(dhp.default_config(batch=batch, ckpt_every=3, cfl_forward=0.0, **kw))
        s.set_store_limit(limit)
        for i in range(batch):
            s.set_sample_schedule(i, sched)
        s.forward(to_gpu(w), 1.0)
        s.loss(to_gpu(t))
        g = s.backward()[0].clone()
        s.close()
        return g

    both = gradient(white, target, 2, 4)
    assert torch.isfinite(both).all() and both[1].abs().max() > 0
    for limit in (-1, 0, 4):
        assert torch.equal(both[1], gradient(white[1], target[1], 1, limit)), limit
