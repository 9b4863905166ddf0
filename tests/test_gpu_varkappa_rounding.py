"""FP32 rounding of the variable-kappa kernels, against FP64 arithmetic on the same
FP32-representable data (RMS over the output, relative to its norm).

Velocity half-step, 1D m = 1 (a series of one term): the interpolant times w_0 and
the term are added by one multiply-add, 3.92e-8 off FP64 over 65536 nodes; rounded
apart they are 4.23e-8 off.  The data sets scatter by 0.3%, the bound lies between."""

import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


def _f32(x):
    return np.float32(x).astype(np.float64)


def _kappa(rng, d, m, K):
    kp, ku = (_f32(0.02 * rng.uniform(-1, 1, tuple(K) + (2 * m + 2,) * d)) for _ in range(2))
    kp[(Ellipsis,) + (0,) * d] = ku[(Ellipsis,) + (0,) * d] = 1.125
    return kp, ku


def _off(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("seed", range(3))
def test_velocity_half_step_of_one_term(seed):
    print(f"[rounding] u half {seed}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(seed)
    K = (1 << 16,)
    P, U = _f32(rng.uniform(-1, 1, K + (2,))), _f32(rng.uniform(-1, 1, (1,) + K + (2,)))
    kp, ku = _kappa(rng, 1, 1, K)
    out = []
    for prec in ("fp64", "fp32"):
        plan = hl.Plan(1, 1, K, length=(K[0] / 64,), cfl=0.45, c=1.2, precision=prec)
        plan.set_kappa(kp, ku)
        p, u = plan.alloc()
        plan.init(p, u, P, U)
        plan.u_half(u, p)
        out.append(plan.export(p, u)[1])
    assert _off(out[1], out[0]) <= 4.07e-8
