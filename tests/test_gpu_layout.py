"""Host layout <-> the stored planes, converted on the device.

The conversion transposes blocks of 32 nodes by 64 coefficients; node counts lie
around a block, coefficient counts reach past one (3D kappa at m = 2: 216).
Storing rounds once: FP64 keeps the value, FP32 is its nearest float, FP32_COMP
holds it to 2^-33 (hi within 2^-24, lo the BF16 rounding of the rest).
"""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


def _stored(x, prec):
    return x.astype(np.float32).astype(np.float64) if prec == "fp32" else x


def _same(got, x, prec):
    if prec == "fp32_comp":
        assert np.all(np.abs(got - x) <= 2.0 ** -33 * np.abs(x))
    else:
        assert np.array_equal(got, _stored(x, prec))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("d,m,K,boundary", [
    (1, 1, (31,), "periodic"), (1, 5, (32,), "walls"), (1, 2, (33,), "periodic"), (1, 3, (1025,), "periodic"),
    (2, 1, (31, 1), "periodic"), (2, 3, (8, 4), "walls"), (2, 5, (11, 3), "periodic"), (2, 2, (65, 33), "walls"),
    (3, 1, (3, 11, 1), "periodic"), (3, 2, (4, 2, 4), "walls"), (3, 3, (5, 7, 3), "periodic"),
])
def test_round_trip(d, m, K, boundary, prec):
    if min(K) < 2:
        K = tuple(max(k, 2) for k in K)
    print(f"[layout] d={d} m={m} K={K} {boundary} {prec}", file=sys.stderr, flush=True)
    plan = hl.Plan(d, m, K, cfl=0.5, precision=prec, boundary=boundary)
    ps, us = plan.host_shapes()
    rng = np.random.default_rng(d + 10 * m)
    P0, U0 = rng.uniform(-1, 1, ps), rng.uniform(-1, 1, us)
    if boundary == "walls":
        P0 = inputs.zero_on_walls(P0, d)
    p, u = plan.alloc()
    plan.init(p, u, P0, U0)
    if prec != "fp32_comp":  # plane a (a_1 fastest), node j (j_1 fastest)
        planes = P0.transpose(tuple(range(2 * d - 1, d - 1, -1)) + tuple(range(d - 1, -1, -1)))
        assert np.array_equal(p.cpu().numpy().astype(np.float64), _stored(planes.reshape(-1), prec))
    P, U = plan.export(p, u)
    _same(P, P0, prec)
    _same(U, U0, prec)


@pytest.mark.parametrize("d,m,K,boundary", [(2, 2, (33, 8), "walls"), (2, 1, (5, 7), "periodic"),
                                            (3, 1, (4, 3, 3), "walls"), (3, 2, (3, 4, 3), "periodic")])
def test_kappa_data_refused_leaves_the_old(d, m, K, boundary):
    print(f"[layout] kappa d={d} m={m} K={K} {boundary}", file=sys.stderr, flush=True)
    plan = hl.Plan(d, m, K, cfl=0.4, c=1.5, precision="fp64", boundary=boundary)
    ps, us = plan.host_shapes()
    rng = np.random.default_rng(m)
    n2 = (2 * m + 2,) * d
    kp, ku = 0.01 * rng.uniform(-1, 1, ps[:d] + n2), 0.01 * rng.uniform(-1, 1, tuple(K) + n2)
    kp[(Ellipsis,) + (0,) * d] = 1.0
    ku[(Ellipsis,) + (0,) * d] = 1.0
    P0 = rng.uniform(-1, 1, ps)
    if boundary == "walls":
        P0 = inputs.zero_on_walls(P0, d)
    U0 = rng.uniform(-1, 1, us)

    def stepped():
        p, u = plan.alloc()
        plan.init(p, u, P0, U0)
        plan.step(p, u, 2)
        return plan.export(p, u)

    plan.set_kappa(kp, ku)
    before = stepped()
    for bad, at in ((kp, -1), (ku, 0)):
        x = bad.copy()
        x.reshape(-1)[at] = np.nan if at else np.inf
        with pytest.raises(hl.HLError):
            plan.set_kappa(x if bad is kp else kp, x if bad is ku else ku)
    after = stepped()
    assert np.array_equal(before[0], after[0]) and np.array_equal(before[1], after[1])
