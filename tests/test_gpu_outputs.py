"""The half-steps' output update and the 3D tiles.

A state larger than the last-level cache whose rows are whole 128-byte lines is
updated with streamed (non-temporal) accesses, a smaller one with cached
accesses; both must store the same values.  The large grid holds a small one
repeated along its last dimension (same spacings and dt), so every copy must
equal the small grid's result bit for bit.

3D workgroups stage tiles of 64 x 4 nodes (two layers in z for the pressure
half-step at m <= 2) plus their upper neighbours: the grids below end just
before, at and just after a tile in every dimension, and wrap inside one tile.
"""

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


@pytest.mark.parametrize("d,m,K,copies,prec", [
    (2, 3, (512, 64), 24, "fp64"),
    (2, 2, (1024, 32), 128, "fp32"),
    (2, 3, (1024, 32), 32, "fp32_comp"),
    (3, 1, (64, 32, 8), 80, "fp64"),
    (3, 2, (64, 20, 9), 60, "fp32"),
    (3, 3, (64, 12, 7), 36, "fp32_comp"),
])
def test_streamed_and_cached_outputs_agree(d, m, K, copies, prec):
    print(f"[outputs] streamed d={d} m={m} K={K} x{copies} {prec}", file=sys.stderr, flush=True)
    big = K[:-1] + (K[-1] * copies,)
    h = 1.0 / max(K)
    length = [k * h for k in K]
    small = hl.Plan(d, m, K, length=length, dt=0.4 * h, precision=prec)
    large = hl.Plan(d, m, big, length=length[:-1] + [length[-1] * copies], dt=0.4 * h, precision=prec)
    bytes_ = (large.info.p_words + large.info.u_words) * large.info.word_bytes
    assert bytes_ > 256 << 20 and big[0] * large.info.word_bytes % 128 == 0
    assert (small.info.p_words + small.info.u_words) * small.info.word_bytes < 256 << 20
    rng = np.random.default_rng(d * 10 + m)
    p, u = small.alloc()
    small.init(p, u, inputs.random_data(rng, d, m, K), inputs.random_data(rng, d, m, K, ncomp=d))

    def repeated(x, fields):  # every plane is its nodes, the last dimension slowest
        words = {"fp64": 1, "fp32": 1, "fp32_comp": 2}[prec]
        if prec == "fp32_comp":  # hi planes (two 16-bit words a value), then lo planes
            nodes = int(np.prod(K))
            n = 2 * fields * nodes
            hi = x[:n].view(fields, 1, words * nodes).expand(-1, copies, -1).reshape(-1)
            lo = x[n:].view(fields, 1, nodes).expand(-1, copies, -1).reshape(-1)
            return torch.cat([hi, lo])
        return x.view(fields, 1, -1).expand(-1, copies, -1).reshape(-1)

    nc = (m + 1) ** d
    P, U = repeated(p, nc).contiguous(), repeated(u, d * nc).contiguous()
    small.step(p, u, 2)
    large.step(P, U, 2)
    torch.cuda.synchronize()
    assert torch.equal(P, repeated(p, nc)) and torch.equal(U, repeated(u, d * nc))


@pytest.mark.parametrize("K", [(2, 2, 2), (3, 2, 5), (63, 3, 3), (64, 4, 2), (65, 5, 3), (129, 2, 2)])
@pytest.mark.parametrize("m,prec,boundary", [(1, "fp64", "periodic"), (2, "fp64", "walls"), (2, "fp32", "periodic"),
                                             (2, "fp32_comp", "periodic"), (3, "fp64", "periodic")])
def test_3d_tiles_match_oracle(m, prec, boundary, K):
    if m == 3 and np.prod(K) > 600:
        K = (65, 3, 3)
    print(f"[outputs] tiles m={m} K={K} {prec} {boundary}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(sum(K) + m)
    plan = hl.Plan(3, m, K, cfl=0.6, precision=prec, boundary=boundary)
    P0 = inputs.random_data(rng, 3, m, plan.host_shapes()[0][:3])
    if boundary == "walls":
        P0 = inputs.zero_on_walls(P0, 3)
    U0 = rng.uniform(-1, 1, plan.host_shapes()[1])
    p, u = plan.alloc()
    plan.init(p, u, P0, U0)
    P_in, U_in = plan.export(p, u)
    prob = oracle.Problem(3, m, K, (1.0,) * 3, plan.dt, 1.0, boundary)
    plan.p_half(p, u)
    Pg, _ = plan.export(p, u)
    _close(Pg, oracle.p_half(prob, P_in, U_in), *tol(prec, 3, m))
    plan.u_half(u, p)
    _, Ug = plan.export(p, u)
    _close(Ug, oracle.u_half(prob, U_in, Pg), *tol(prec, 3, m))
