"""1D multi-step launches: hl_step on a constant-coefficient 1D plan runs many
steps per launch (one workgroup holding the grid, or workgroups with a halo),
and must leave exactly what stepping half-step by half-step leaves, ghost nodes
included.  Sizes around the one-workgroup limit (768 nodes), the owned stretch
(256) and the halo (32 steps)."""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("boundary", ["periodic", "walls"])
@pytest.mark.parametrize("m,K", [(1, 2), (3, 3), (1, 200), (0, 767), (1, 768), (1, 769), (7, 511), (7, 513), (2, 1023),
                                 (3, 1025), (1, 5000)])
def test_multi_step_launches_equal_half_steps(m, K, boundary, prec):
    print(f"[steps1d] m={m} K={K} {boundary} {prec}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(m + K)
    plan = hl.Plan(1, m, (K,), cfl=0.6, precision=prec, boundary=boundary)
    P0 = inputs.random_data(rng, 1, m, plan.host_shapes()[0][:1])
    if boundary == "walls":
        P0 = inputs.zero_on_walls(P0, 1)
    p, u = plan.alloc()
    plan.init(p, u, P0, rng.uniform(-1, 1, plan.host_shapes()[1]))
    q, v = p.clone(), u.clone()
    for n in (1, 4, 33, 70):
        plan.step(p, u, n)
        for _ in range(n):
            plan.p_half(q, v)
            plan.u_half(v, q)
        torch.cuda.synchronize()
        assert torch.equal(p, q) and torch.equal(u, v), n


def test_two_streams_share_a_plan():
    """Two states stepped on two streams by one plan of several workgroups."""
    print("[steps1d] two streams", file=sys.stderr, flush=True)
    rng = np.random.default_rng(9)
    plan = hl.Plan(1, 2, (3000,), cfl=0.5, precision="fp64")
    states = []
    for _ in range(2):
        p, u = plan.alloc()
        plan.init(p, u, inputs.random_data(rng, 1, 2, (3000,)), inputs.random_data(rng, 1, 2, (3000,), ncomp=1))
        states.append((p, u, p.clone(), u.clone()))
    streams = [torch.cuda.Stream() for _ in states]
    torch.cuda.synchronize()
    for _ in range(5):
        for s, (p, u, _, _) in zip(streams, states):
            plan.step(p, u, 40, stream=s)
    torch.cuda.synchronize()
    for p, u, q, v in states:
        for _ in range(200):
            plan.p_half(q, v)
            plan.u_half(v, q)
        torch.cuda.synchronize()
        assert torch.equal(p, q) and torch.equal(u, v)
