"""Host layout conversion at the limits of one launch and one staging buffer.

A slab launch has one workgroup of 256 work-items per row (j_2, j_3) and 32 j_1,
and fewer than 2^32 work-items: at 2^24 - 1 rows the device converts, at 2^24
the host does."""

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
