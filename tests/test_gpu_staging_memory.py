"""Device memory of the host-layout staging: one buffer of at most 64 MB per GPU,
whatever the number of plans, given back with the last plan; calls on several
plans from several threads at once are right."""

import gc
import sys
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402

MB = 1 << 20


def _used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_one_buffer_for_all_plans():
    print("[staging] one buffer", file=sys.stderr, flush=True)
    gc.collect()  # plans of earlier tests
    K, m = (1000, 400), 3  # 51 MB per component in host layout
    plans = [hl.Plan(2, m, K, precision="fp32") for _ in range(8)]
    states = [plan.alloc() for plan in plans]
    P = np.ones(plans[0].host_shapes()[0])
    for p, u in states:
        p.zero_()
        u.zero_()
    before = _used()
    for plan, (p, u) in zip(plans, states):
        plan.init(p, u, P)
    assert _used() - before <= 64 * MB + 16 * MB  # the buffer, and the allocator's granularity
    for plan in plans:
        plan.close()
    gc.collect()
    assert _used() - before <= 16 * MB


def test_threads_share_the_buffer():
    print("[staging] threads", file=sys.stderr, flush=True)
    rng = np.random.default_rng(2)
    work, failed = [], []
    for i in range(6):
        K = (200 + 13 * i, 150)
        plan = hl.Plan(2, 2, K, precision="fp64")
        ps, us = plan.host_shapes()
        work.append((plan, plan.alloc(), rng.uniform(-1, 1, ps), rng.uniform(-1, 1, us), torch.cuda.Stream()))
    torch.cuda.synchronize()

    def run(plan, state, P, U, stream):
        try:
            for _ in range(8):
                plan.init(*state, P, U, stream=stream)
                P2, U2 = plan.export(*state, stream=stream)
                assert np.array_equal(P, P2) and np.array_equal(U, U2)
        except BaseException as e:  # noqa: BLE001
            failed.append(e)

    threads = [threading.Thread(target=run, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
