"""What a handle does after a call has failed half-way, on a stand-in for the HIP runtime
(tests/hip_stub.cpp, preloaded into a child process): kernels do nothing, chosen runtime calls
fail, and the stand-in keeps watch over what the library asks of it.  No GPU needed."""

import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2502_02294_amd", "libdiffhydro.so")

PRELUDE = """
import ctypes, importlib.util, sys
spec = importlib.util.spec_from_file_location("binding", sys.argv[1])
b = importlib.util.module_from_spec(spec)
spec.loader.exec_module(b)
lib, stub = b.lib(), ctypes.CDLL(None)
stub.stub_log.restype = ctypes.c_char_p
def create(**kw):
    c = b.Config()
    lib.dh_config_default(ctypes.byref(c))
    c.n, c.box = 16, 2.5
    for k, v in kw.items():
        setattr(c, k, v)
    h = ctypes.c_void_p()
    assert lib.dh_create(ctypes.byref(c), ctypes.byref(h)) == 0
    return h
def buf(count):
    return ctypes.cast((ctypes.c_float * count)(*[0.5] * count), ctypes.c_void_p)
N = ctypes.c_int32()
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(LIB):
        from paper_2502_02294_amd import build_lib
        build_lib.build(verbose=False)
    so = tmp_path_factory.mktemp("stub") / "hip_stub.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                    os.path.join(HERE, "hip_stub.cpp"), "-o", str(so)], check=True)
    return str(so)


def run(stub, code, *args):
    env = dict(os.environ)
    env["LD_PRELOAD"] = ":".join(p for p in (stub, env.get("LD_PRELOAD")) if p)
    binding = os.path.join(ROOT, "paper_2502_02294_amd", "_lib.py")
    r = subprocess.run([sys.executable, "-c", PRELUDE + code, binding, *map(str, args)], env=env,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


@pytest.mark.parametrize("kernel", ["kick_drift_kernel", "sweep_x_kernel", "scan_kernel",
                                    "scatter_kernel", "bin_sort_gather_kernel",
                                    "bin_sort_large_kernel", "deposit_kernel"])
def test_bin_counts_are_clear_after_a_failed_step(stub, kernel):
    """A step counts the particles' bins in the drift and clears the counts in the sort; a
    histogram on counts that a failed call left behind would index past the particles."""
    run(stub, """
h = create()
pos, rho, out = buf(3 * 16**3), buf(16**3), buf(16**3)
assert lib.dh_init_from_seed(h, 1) == 0
for again in (lambda: lib.dh_run_steps(h, 1, ctypes.byref(N)),
              lambda: lib.dh_stage_deposit(h, rho, pos, out),
              lambda: lib.dh_init_from_seed(h, 2)):
    stub.stub_fail_kernel(sys.argv[2].encode())
    assert lib.dh_run_steps(h, 1, ctypes.byref(N)) == -3
    assert again() == 0
    assert lib.dh_init_from_seed(h, 1) == 0
    assert lib.dh_run_steps(h, 2, ctypes.byref(N)) == 0
    assert stub.stub_dirty_counts() == 0, sys.argv[2]
""", kernel)


@pytest.mark.parametrize("kind", ["malloc", "host_malloc"])
@pytest.mark.parametrize("call", ["backward", "forward", "fli_loss", "power_loss"])
def test_a_call_whose_allocation_failed_can_be_made_again(stub, kind, call):
    """Every allocation of a call fails in turn; the call reports it, and made again it works on
    whole buffers: nothing is launched on, or copied through, one that was never allocated."""
    run(stub, """
kind, call = sys.argv[2], sys.argv[3]
white, out, a, c = buf(16**3), buf(16**3), buf(16**3), buf(16**3)
loss, par = (ctypes.c_double * 1)(), (ctypes.c_double * 4)()
pk, sig = (ctypes.c_double * 8)(*[1.0] * 8), (ctypes.c_double * 8)(*[1.0] * 8)
fail = getattr(stub, "stub_fail_" + kind)
fails = 0
for k in range(200):
    h = create(ckpt_every=3)
    lib.dh_set_store_limit(h, 3)     # taped steps, checkpoints and recomputed steps
    sched = (ctypes.c_double * 80)(*[1e-4] * 80)
    def forward(steps):
        assert lib.dh_set_schedule(h, sched, steps) == 0
        return lib.dh_forward(h, white, 1.0, ctypes.byref(N))
    if call != "forward":
        assert forward(7) == 0
        assert lib.dh_loss(h, a, loss) == 0
    f = {"backward": lambda: lib.dh_backward(h, None, out, par),
         "forward": lambda: forward(70),
         "fli_loss": lambda: lib.dh_fli_loss(h, a, c, white, loss),
         "power_loss": lambda: lib.dh_power_loss(h, 8, pk, sig, loss)}[call]
    fail(k)
    rc = f()
    fail(-1)
    if rc == 0:
        break
    assert rc in (-2, -3), rc
    fails += 1
    assert f() == 0, (k, lib.dh_last_error(h))
    if call != "backward":
        assert call == "forward" or lib.dh_backward(h, None, out, par) == 0
    else:   # a later, longer run grows the same buffers
        assert forward(70) == 0 and lib.dh_loss(h, a, loss) == 0
        assert f() == 0
    assert stub.stub_null_writes() == 0, k
    assert lib.dh_destroy(h) == 0
assert k < 199 and (fails > 0 or kind == "host_malloc" or call == "power_loss"), (k, fails)
""", kind, call)


def test_a_long_wait_does_not_hold_the_processor(stub):
    """Values handed to the host are watched for a short while; behind work that takes longer
    (a replayed forward is queued as a whole) the wait is the runtime's."""
    run(stub, """
import time
h = create()
loss, a = (ctypes.c_double * 1)(), buf(16**3)
assert lib.dh_init_from_seed(h, 1) == 0
stub.stub_late_values(500)
wall, cpu = time.perf_counter(), time.process_time()
assert lib.dh_loss(h, a, loss) == 0
wall, cpu = time.perf_counter() - wall, time.process_time() - cpu
assert loss[0] * 16**3 == 1.0
assert wall > 0.45 and cpu < 0.2, (wall, cpu)
""")


def test_a_value_that_does_not_arrive_is_an_error(stub):
    run(stub, """
h = create()
loss, a = (ctypes.c_double * 1)(7.0), buf(16**3)
assert lib.dh_init_from_seed(h, 1) == 0
stub.stub_hold_values(1)
assert lib.dh_loss(h, a, loss) == -3
assert loss[0] == 7.0
stub.stub_hold_values(0)
assert lib.dh_loss(h, a, loss) == 0 and loss[0] * 16**3 == 1.0
""")
