"""1D multi-step launches of one plan from calls whose stream handles are equal
but name different streams: the per-thread default stream (one handle, a stream
per host thread), and a destroyed stream's handle given to a new stream.  The
plan's second buffers are shared, so the second call has to wait for the first
one's launches; both states must be what half-steps on another plan leave."""

import ctypes
import sys
import threading
import types

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402

PER_THREAD = types.SimpleNamespace(cuda_stream=2)  # hipStreamPerThread
K, STEPS = (3000,), 640


def _states(plan):
    rng = np.random.default_rng(17)
    out = []
    for _ in range(2):
        p, u = plan.alloc()
        plan.init(p, u, inputs.random_data(rng, 1, 2, K), inputs.random_data(rng, 1, 2, K, ncomp=1))
        out.append((p, u, p.clone(), u.clone()))
    torch.cuda.synchronize()
    return out


def _check(states):
    torch.cuda.synchronize()
    ref = hl.Plan(1, 2, K, cfl=0.5, precision="fp64")
    for p, u, q, v in states:
        for _ in range(STEPS):
            ref.p_half(q, v)
            ref.u_half(v, q)
        torch.cuda.synchronize()
        assert torch.equal(p, q) and torch.equal(u, v)


def test_per_thread_streams():
    print("[steps1d] per-thread default streams", file=sys.stderr, flush=True)
    plan = hl.Plan(1, 2, K, cfl=0.5, precision="fp64")
    states = _states(plan)
    launched, done = [threading.Event() for _ in states], threading.Event()
    failed = []

    def run(i):
        try:
            if i:
                launched[i - 1].wait(60)
            p, u = states[i][:2]
            plan.step(p, u, STEPS, stream=PER_THREAD)
        except Exception as e:  # noqa: BLE001
            failed.append(e)
        launched[i].set()
        done.wait(60)  # both threads, and so both streams, live until all is launched

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for e in launched:
        assert e.wait(60)
    done.set()
    for t in threads:
        t.join()
    assert not failed, failed
    _check(states)


def test_stream_handle_given_again():
    print("[steps1d] a stream after another", file=sys.stderr, flush=True)
    with open("/proc/self/maps") as maps:  # the HIP runtime this process runs
        paths = {line.split()[-1] for line in maps if "libamdhip64" in line}
    assert len(paths) == 1, paths
    hip = ctypes.CDLL(paths.pop())
    hip.hipStreamCreateWithFlags.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint]
    hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    plan = hl.Plan(1, 2, K, cfl=0.5, precision="fp64")
    states = _states(plan)
    for p, u, _, _ in states:
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0  # non-blocking
        plan.step(p, u, STEPS, stream=types.SimpleNamespace(cuda_stream=s.value))
        assert hip.hipStreamDestroy(s) == 0
    _check(states)
