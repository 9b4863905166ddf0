"""Host layout conversion at the limits of one launch and one staging buffer.

A slab launch has one workgroup of 256 work-items per row (j_2, j_3) and 32 j_1,
and fewer than 2^32 work-items: at 2^24 - 1 rows the device converts, at 2^24
the host does.  A component crosses through the shared staging buffer (64 MB), a
temporary one (256 MB), or in slabs of j_1; what has no slab, the host converts."""

import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


def _round_trip(d, m, K):
    """p and the first velocity component against the planes of their layout,
    and back."""
    plan = hl.Plan(d, m, K, length=[k / max(K) for k in K], cfl=0.5, precision="fp64")
    ps, us = plan.host_shapes()
    nodes, nc = int(np.prod(K)), (m + 1) ** d
    P = np.arange(nodes * nc, dtype=np.float64).reshape(ps)
    U = np.arange(d * nodes * nc, dtype=np.float64).reshape(us)
    U *= -0.5
    p, u = plan.alloc()
    plan.init(p, u, P, U)
    order = tuple(range(2 * d - 1, d - 1, -1)) + tuple(range(d - 1, -1, -1))  # planes a, nodes j, first index fastest
    host = torch.from_numpy(P)
    assert torch.equal(p, host.cuda().permute(order).reshape(-1))
    assert torch.equal(u[:nodes * nc], torch.from_numpy(U[0]).cuda().permute(order).reshape(-1))
    P2, U2 = plan.export(p, u)
    assert np.array_equal(P2, P) and np.array_equal(U2, U)


@pytest.mark.parametrize("rows", [2 ** 24 - 1, 2 ** 24])
def test_rows_at_the_launch_limit(rows):
    print(f"[layout] 2 x {rows} m=0", file=sys.stderr, flush=True)
    _round_trip(2, 0, (2, rows))


@pytest.mark.parametrize("d,m,K", [
    (2, 3, (1031, 700)),     # 92 MB per component: past the shared staging buffer
    (2, 3, (1451, 1500)),    # 279 MB: two slabs, the last of 53 of 1398 j_1
    (1, 7, (4300001,)),      # 275 MB: two slabs, the last ending inside a block
])
def test_components_past_the_staging_buffers(d, m, K):
    print(f"[layout] d={d} m={m} K={K}", file=sys.stderr, flush=True)
    _round_trip(d, m, K)


@pytest.mark.parametrize("d,m,K,copies", [
    (1, 7, (11,), 100003),      # both kappa arrays together past the staged check: each converted by itself
    (2, 1, (2, 21), 100000),    # one j_1 of kappa data past a slab: converted on the host
])
def test_kappa_data_past_the_staging_buffers(d, m, K, copies):
    """A grid that repeats a small one along its last dimension, with its spacing
    and dt, gives the small grid's result in every copy."""
    print(f"[layout] kappa d={d} m={m} K={K} x{copies}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(m)
    big = K[:-1] + (K[-1] * copies,)
    length = [float(k) for k in K]
    n2 = (2 * m + 2,) * d
    kp, ku = (0.01 * rng.uniform(-1, 1, K + n2) for _ in range(2))
    kp[(Ellipsis,) + (0,) * d] = ku[(Ellipsis,) + (0,) * d] = 1.0
    fields = [rng.uniform(-1, 1, lead + K + (m + 1,) * d) for lead in ((), (d,), (), (d,))]

    def repeated(x, axis):
        return np.tile(x, [copies if a == axis else 1 for a in range(x.ndim)])

    def run(K, length, kp, ku, fields):
        plan = hl.Plan(d, m, K, length=length, dt=0.4, c=1.2, precision="fp64")
        plan.set_kappa(kp, ku)
        (p, u), (pb, ub) = plan.alloc(), plan.alloc()
        plan.init(p, u, *fields[:2])
        plan.init(pb, ub, *fields[2:])
        plan.step(p, u, 2)
        plan.adjoint_step_var(pb, ub, p, u)
        out = list(plan.export(p, u)) + list(plan.kappa_grad(reset=True))
        plan.close()
        return out

    small = run(K, length, kp, ku, fields)
    large = run(big, length[:-1] + [length[-1] * copies], repeated(kp, d - 1), repeated(ku, d - 1),
                [repeated(f, d - 1 + (i % 2)) for i, f in enumerate(fields)])
    for i, (a, b) in enumerate(zip(small, large)):
        assert np.array_equal(repeated(a, d if i == 1 else d - 1), b), i
