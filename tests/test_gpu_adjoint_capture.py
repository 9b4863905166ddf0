"""The kappa gradient under stream capture: once a plan has computed a gradient,
a further call allocates nothing, also after hl_set_tile has given it more
workgroups than before.  Every replay must leave what the same eager call
leaves."""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


@pytest.mark.parametrize("d,m,K,tile,boundary", [(1, 3, (5000,), (64, 1), "periodic"),
                                                 (2, 2, (300, 37), (32, 2), "periodic"),
                                                 (2, 1, (129, 66), (64, 1), "walls"),
                                                 (3, 1, (70, 9, 6), (96, 1), "periodic")])
def test_captured_gradient_with_smaller_tiles(d, m, K, tile, boundary):
    print(f"[capture] d={d} m={m} K={K} {tile} {boundary}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(3 * d + m)
    plan = hl.Plan(d, m, K, cfl=0.5, precision="fp64", boundary=boundary)
    ps, us = plan.host_shapes()

    def field():
        P = rng.uniform(-1, 1, ps)
        p, u = plan.alloc()
        plan.init(p, u, inputs.zero_on_walls(P, d) if boundary == "walls" else P, rng.uniform(-1, 1, us))
        return p, u

    p, u = field()
    pb0, ub0 = field()
    g = torch.zeros(1, dtype=torch.float64, device="cuda")
    pb, ub = pb0.clone(), ub0.clone()
    plan.adjoint_step(pb, ub, 2, p=p, u=u, grad_kappa=g)  # allocates
    plan.set_tile(*tile)
    eager = []
    pb, ub = pb0.clone(), ub0.clone()
    g.zero_()
    for _ in range(3):
        plan.adjoint_step(pb, ub, 2, p=p, u=u, grad_kappa=g)
        eager.append((pb.clone(), ub.clone(), g.clone()))
    assert bool(eager[-1][2] != 0)
    pb.copy_(pb0)
    ub.copy_(ub0)
    g.zero_()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.adjoint_step(pb, ub, 2, p=p, u=u, grad_kappa=g)
    for ref in eager:
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip((pb, ub, g), ref):
            assert torch.equal(got, want)
        plan.step(p.clone(), u.clone(), 1)  # the program's own work between replays
