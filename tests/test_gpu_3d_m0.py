"""3D m = 0: the half-steps, the transposed half-steps and the gradient's inner
products load a node's corners directly (no staging).  Against the oracle at the
edges of a tile in every dimension, periodic and walls, and batched shots
against their plans' own steps."""

import sys

import numpy as np
import pytest

import oracle
from paper_1808_10481_amd import inputs
from tolerances import _close, tol

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402

SIZES = [(2, 2, 2), (3, 5, 2), (63, 3, 3), (64, 4, 2), (65, 9, 3), (129, 2, 2)]


def _fields(plan, boundary, rng):
    ps, us = plan.host_shapes()
    P = rng.uniform(-1, 1, ps)
    return inputs.zero_on_walls(P, 3) if boundary == "walls" else P, rng.uniform(-1, 1, us)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("boundary", ["periodic", "walls"])
@pytest.mark.parametrize("K", SIZES)
def test_half_steps_and_adjoint(K, boundary, prec):
    print(f"[3d m0] {K} {boundary} {prec}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(sum(K))
    plan = hl.Plan(3, 0, K, cfl=0.6, c=1.2, precision=prec, boundary=boundary)
    prob = oracle.Problem(3, 0, K, (1.0,) * 3, plan.dt, plan.kappa, boundary)
    p, u = plan.alloc()
    plan.init(p, u, *_fields(plan, boundary, rng))
    P0, U0 = plan.export(p, u)
    plan.p_half(p, u)
    P1, _ = plan.export(p, u)
    _close(P1, oracle.p_half(prob, P0, U0), *tol(prec, 3, 0))
    plan.u_half(u, p)
    _, U1 = plan.export(p, u)
    _close(U1, oracle.u_half(prob, U0, P1), *tol(prec, 3, 0))
    # the transposed step: two half-steps, each within the forward bound
    pb, ub = plan.alloc()
    plan.init(pb, ub, *_fields(plan, "periodic", rng))
    Pb, Ub = plan.export(pb, ub)
    plan.adjoint_step(pb, ub, 1)
    Pg, Ug = plan.export(pb, ub)
    Pr, Ur = oracle.adjoint_step(prob, Pb, Ub, 1)
    l2, mx = tol(prec, 3, 0)
    _close(Pg, Pr, 2 * l2, 2 * mx)
    _close(Ug, Ur, 2 * l2, 2 * mx)


@pytest.mark.parametrize("tile", [(0, 0), (32, 5), (96, 2), (256, 1)])
@pytest.mark.parametrize("K", [(3, 5, 2), (65, 9, 3)])
def test_gradient(K, tile):
    """FP64: n products per node in sums of one sign pattern, 1e-9 relative as
    for the other orders."""
    print(f"[3d m0] gradient {K} {tile}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(sum(K) + 1)
    plan = hl.Plan(3, 0, K, cfl=0.7, c=1.1, precision="fp64")
    plan.set_tile(*tile)
    prob = oracle.Problem(3, 0, K, (1.0,) * 3, plan.dt, plan.kappa)
    (p, u), (pb, ub) = plan.alloc(), plan.alloc()
    plan.init(p, u, *_fields(plan, "periodic", rng))
    plan.init(pb, ub, *_fields(plan, "periodic", rng))
    P0, U0 = plan.export(p, u)
    Pb, Ub = plan.export(pb, ub)
    plan.step(p, u, 3)
    g = torch.zeros(1, dtype=torch.float64, device="cuda")
    plan.adjoint_step(pb, ub, 3, p=p, u=u, grad_kappa=g)
    gr, Pr, Ur = oracle.kappa_gradient(prob, P0, U0, Pb, Ub, 3)
    assert abs(float(g) - gr) <= 1e-9 * abs(gr), (float(g), gr)
    Pa, Ua = plan.export(pb, ub)
    _close(Pa, Pr, 6e-12, 6e-11)
    _close(Ua, Ur, 6e-12, 6e-11)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_comp"])
def test_batch(prec):
    print(f"[3d m0] batch {prec}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(4)
    plans, states = [], []
    for K, boundary in zip(SIZES, ["periodic", "walls"] * 3):
        plan = hl.Plan(3, 0, K, cfl=0.6, precision=prec, boundary=boundary)
        p, u = plan.alloc()
        plan.init(p, u, *_fields(plan, boundary, rng))
        plans.append(plan)
        states.append((p, u, p.clone(), u.clone()))
    batch = hl.Batch(plans)
    batch.step([s[0] for s in states], [s[1] for s in states], 19)
    for plan, (_, _, q, v) in zip(plans, states):
        plan.step(q, v, 19)
    torch.cuda.synchronize()
    for p, u, q, v in states:
        assert torch.equal(p, q) and torch.equal(u, v)
