"""The kappa-data gradient's accumulators and the adjoint's scratch arrays are
cleared on the null stream, which non-blocking streams (torch's side streams)
do not wait for; the calls that clear them return only when they are clear, so
a gradient on a side stream has the value it has on the default stream."""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import autograd as hag  # noqa: E402
from paper_1808_10481_amd import hl  # noqa: E402


@pytest.mark.parametrize("m,K,boundary", [(2, (192, 160), "periodic"), (1, (96, 65), "walls")])
def test_traces_gradient_on_a_side_stream(m, K, boundary):
    print(f"[kstreams] traces m={m} K={K} {boundary}", file=sys.stderr, flush=True)
    d = 2
    rng = np.random.default_rng(31 + m)
    grads = []
    shapes = None
    for side in (False, True, True):
        plan = hl.Plan(d, m, K, cfl=0.4, c=1.5, precision="fp64", boundary=boundary)
        ps, us = plan.host_shapes()
        if shapes is None:
            n2 = (2 * m + 2,) * d
            kp, ku = 0.01 * rng.uniform(-1, 1, ps[:d] + n2), 0.01 * rng.uniform(-1, 1, tuple(K) + n2)
            kp[(Ellipsis,) + (0,) * d] = 1.5
            ku[(Ellipsis,) + (0,) * d] = 1.5
            P = rng.uniform(-1, 1, ps)
            P = inputs.zero_on_walls(P, d) if boundary == "walls" else P
            shapes = ps, us
        p, u = plan.alloc()
        plan.init(p, u, P, np.zeros(us))
        torch.cuda.synchronize()
        stream = torch.cuda.Stream() if side else torch.cuda.current_stream()
        with torch.cuda.stream(stream):
            for _ in range(2):  # the second backward finds the accumulators used and reset
                kpt = torch.tensor(kp, requires_grad=True)
                kut = torch.tensor(ku, requires_grad=True)
                tr, _, _ = hag.receiver_traces(kpt, kut, p, u, plan, 6, [(3, 5), (40, 31), (K[0] - 1, K[1] - 2)])
                (tr ** 2).sum().backward()
                grads.append((kpt.grad.numpy(), kut.grad.numpy()))
        torch.cuda.synchronize()
    for gp, gu in grads[1:]:
        assert np.array_equal(gp, grads[0][0]) and np.array_equal(gu, grads[0][1])


@pytest.mark.parametrize("d,m,K", [(2, 3, (130, 90)), (3, 1, (40, 33, 18))])
def test_walled_adjoint_on_a_side_stream(d, m, K):
    print(f"[kstreams] walled adjoint d={d} m={m} K={K}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(d)
    out = []
    for side in (False, True):
        plan = hl.Plan(d, m, K, cfl=0.4, precision="fp64", boundary="walls")
        ps, us = plan.host_shapes()
        if not out:
            P, U = inputs.zero_on_walls(rng.uniform(-1, 1, ps), d), rng.uniform(-1, 1, us)
        pb, ub = plan.alloc()
        plan.init(pb, ub, P, U)
        torch.cuda.synchronize()
        stream = torch.cuda.Stream() if side else torch.cuda.current_stream()
        plan.adjoint_step(pb, ub, 3, stream=stream)
        torch.cuda.synchronize()
        out.append((pb, ub))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
