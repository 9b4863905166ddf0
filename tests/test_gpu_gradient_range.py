"""The kappa gradient at the end of FP64's range: a product that overflows makes
the sum infinite with its sign (a plain sum's value), not NaN.

One adjoint velocity entry is nonzero, so the velocity side of one step is the
single product -<u_bar, B_kappa P'> (terms of zero adjoint entries are zero);
p_bar is chosen so that p_bar - B^T u_bar is zero in every bit, which makes the
pressure side zero.  Scaling u_bar and p by 1e200 each makes the product
overflow; its sign is that of the unscaled gradient."""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


@pytest.mark.parametrize("boundary", ["periodic", "walls"])
@pytest.mark.parametrize("d,m,K", [(1, 2, (70,)), (2, 2, (66, 5)), (3, 1, (65, 5, 3)), (3, 2, (9, 5, 3))])
def test_overflowing_gradient_is_infinite(d, m, K, boundary):
    print(f"[range] d={d} m={m} K={K} {boundary}", file=sys.stderr, flush=True)
    plan = hl.Plan(d, m, K, cfl=0.5, precision="fp64", boundary=boundary)
    rng = np.random.default_rng(5 + d)
    ps, us = plan.host_shapes()
    P = rng.uniform(0.5, 1, ps)
    if boundary == "walls":
        P = inputs.zero_on_walls(P, d)

    def gradient(scale, entry):
        p, u = plan.alloc()
        plan.init(p, u, P * scale, np.zeros(us))
        U = np.zeros(us)
        U.reshape(-1)[entry] = scale
        pb, ub = plan.alloc()
        plan.init(pb, ub, np.zeros(ps), U)
        q, v = pb.clone(), ub.clone()
        plan.adjoint_step(q, v, 1)   # q = 0 - B^T u_bar
        pb = -q
        g = torch.zeros(1, dtype=torch.float64, device="cuda")
        plan.adjoint_step(pb, ub, 1, p=p, u=u, grad_kappa=g)
        assert not pb.any()
        return float(g)

    for entry in (3 * (m + 1) ** d, 3 * (m + 1) ** d + 1):
        g1 = gradient(1.0, entry)
        assert np.isfinite(g1) and g1 != 0.0
        assert gradient(1e200, entry) == np.copysign(np.inf, g1)
