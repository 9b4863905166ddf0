"""1D transposed half-steps in FP32 round no more than the plain evaluation: each
corner's data times its block entry, one multiply-add at a time in FP32, from the
oracle's blocks.  Both errors are taken against FP64 on the same inputs and
blocks.  Over 4096 nodes or more values the ratio of two independent RMS errors
of one size scatters by less than 1 / sqrt(2 * 4096) = 1.1%; the bound is five
times that."""

import sys

import numpy as np
import pytest

import oracle
from oracle import hermite_lf

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402

K = 4096


def _minus_blocks(x, blocks, y, first, prec):
    """x[j] - sum_e sum_c blocks[e][:, c] y[j + first + e][c], summed corner by
    corner in prec."""
    acc = np.zeros_like(x)
    for e in range(2):
        src = np.roll(y, -(first + e), axis=0)
        for c in range(y.shape[1]):
            acc = (acc + blocks[e][:, c].astype(prec).astype(np.float64) * src[:, c:c + 1]).astype(prec).astype(np.float64)
    return (x - acc).astype(prec).astype(np.float64)


@pytest.mark.parametrize("m", range(8))
def test_rounding_of_the_1d_adjoint(m):
    print(f"[adjoint 1d] m={m}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(m)
    plan = hl.Plan(1, m, (K,), cfl=0.6, c=1.2, precision="fp32")
    prob = oracle.Problem(1, m, (K,), (1.0,), plan.dt, plan.kappa)
    pb, ub = plan.alloc()
    plan.init(pb, ub, rng.uniform(-1, 1, (K, m + 1)), rng.uniform(-1, 1, (1, K, m + 1)))
    P, U = plan.export(pb, ub)
    plan.adjoint_step(pb, ub, 1)
    Pg, Ug = plan.export(pb, ub)
    A, B = hermite_lf.p_operator_blocks(prob), hermite_lf.u_operator_blocks(prob)
    # corner e of the gather reads the forward operator's block 1 - e, transposed
    bt = [B[1 - e, 0].T for e in range(2)]
    at = [A[1 - e, :, 0, :].T for e in range(2)]
    for got, x, blocks, y, first in ((Pg, P, bt, U[0], -1), (Ug[0], U[0], at, Pg, 0)):
        exact = _minus_blocks(x, blocks, y, first, np.float64)
        plain = _minus_blocks(x, blocks, y, first, np.float32)
        e_got, e_plain = (np.sqrt(np.mean((v - exact) ** 2)) for v in (got, plain))
        assert e_got <= 1.055 * e_plain, (e_got, e_plain)
