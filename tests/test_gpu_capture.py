"""Stage calls under graph capture.  A call whose table is already on the device is captured; one
that would have to upload its table is refused, as is every call that waits for the device: a
captured upload would not have run, while the handle takes its table for present."""

import pytest
import torch

import synth_inputs as si
from gpu_helpers import to_gpu
from paper_2502_02294_amd._lib import DiffHydroError

pytestmark = pytest.mark.gpu


def _state(dhp, n):
    s = dhp.Sim(dhp.default_config(n=n, box=n * 10.0 / 64, subgrid=0))
    s.init_from_noise(to_gpu(si.white_noise(n, 3)))
    return s, s.get("q").clone()


@pytest.mark.parametrize("n", [16, 32])
def test_upload_under_capture_is_refused(n):
    import paper_2502_02294_amd as dhp
    print(f"capture: upload, n {n}", flush=True)
    s, q = _state(dhp, n)
    want = s.stage_sweep(q, 1, 0.2, 0.02, 0.021).clone()
    s.stage_sweep(q, 1, 0.1, 0.02, 0.021)   # another table on the device
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        g = torch.cuda.CUDAGraph()
        g.capture_begin()
        refused = False
        try:
            s.stage_sweep(q, 1, 0.2, 0.02, 0.021)
        except DiffHydroError:
            refused = True
        finally:
            g.capture_end()
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(s.stage_sweep(q, 1, 0.2, 0.02, 0.021), want)
    assert refused
    s.close()


@pytest.mark.parametrize("n", [16, 32])
def test_captured_stage_replays(n):
    import paper_2502_02294_amd as dhp
    print(f"capture: replays, n {n}", flush=True)
    s, q = _state(dhp, n)
    src = q.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        s.stage_sweep(src, 2, 0.2, 0.02, 0.021)
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        g.capture_begin()
        try:
            out = s.stage_sweep(src, 2, 0.2, 0.02, 0.021)
        finally:
            g.capture_end()
        for k in range(3):
            src.copy_(q)
            src[0].mul_(1.0 + 0.1 * k)
            g.replay()
            side.synchronize()
            assert torch.equal(out, s.stage_sweep(src, 2, 0.2, 0.02, 0.021)), k
    torch.cuda.current_stream().wait_stream(side)
    s.close()
