"""FP32 rounding of the variable-kappa kernels, against FP64 arithmetic on the same
FP32-representable data (RMS over the output, relative to its norm).

Velocity half-step, 1D m = 1 (a series of one term): the interpolant times w_0 and
the term are added by one multiply-add, 3.92e-8 off FP64 over 65536 nodes; rounded
apart they are 4.23e-8 off.  The data sets scatter by 0.3%, the bound lies between.

Gradient with respect to the kappa data: the recurrence's terms fall with k, and a
sum that takes them largest first rounds every later product at the size of the
sum (velocity side, 3D m = 1: 2.4e-7 off instead of 1.62e-7).  The bounds are 1.03
times the mean error, over the three data sets, of summing them smallest first;
the data sets scatter by 1%."""

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


@pytest.mark.parametrize("d,m,K,means", [(3, 1, (32, 24, 20), (2.210e-7, 1.619e-7)),
                                         (2, 2, (96, 80), (2.512e-7, 1.423e-7)),
                                         (2, 1, (128, 100), (1.401e-7, 0.949e-7)),
                                         (1, 2, (8192,), (1.491e-7, 0.814e-7))])
def test_kappa_gradient(d, m, K, means):
    print(f"[rounding] kappa gradient d={d} m={m}", file=sys.stderr, flush=True)
    errs = []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        sh = tuple(K) + (m + 1,) * d
        data = [_f32(rng.uniform(-1, 1, s)) for s in (sh, (d,) + sh, sh, (d,) + sh)]
        kp, ku = _kappa(rng, d, m, K)
        out = []
        for prec in ("fp64", "fp32"):
            plan = hl.Plan(d, m, K, cfl=0.45, c=1.2, precision=prec)
            plan.set_kappa(kp, ku)
            (p, u), (a, b) = plan.alloc(), plan.alloc()
            plan.init(p, u, *data[:2])
            plan.init(a, b, *data[2:])
            plan.adjoint_step_var(a, b, p, u)
            out.append(plan.kappa_grad(reset=True))
        errs.append([_off(x, y) for y, x in zip(*out)])
    for err, mean in zip(np.mean(errs, axis=0), means):
        assert err <= 1.03 * mean, (err, mean)
