"""The two-layer form of the 3D pressure half-step (m = 1, 2): a workgroup's tile
has two node layers in z, from 512 such tiles on.  Its results must equal the
one-layer form's (a tile the layered form does not hold), bit for bit, with a
ragged last tile in x and y and an odd last layer, for the pressure half-step and
for the transposed one, which runs the same kernel.  128 x 2 tiles stage 1161
words for two layers, more than the layered form's 1024."""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


def _layered_tiles(n):
    return -(-n[0] // 64) * -(-n[1] // 4) * -(-n[2] // 2)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("K,boundary", [((65, 9, 171), "periodic"), ((64, 8, 512), "periodic"), ((65, 9, 170), "periodic"),
                                        ((64, 8, 170), "walls"), ((63, 11, 401), "walls")])
@pytest.mark.parametrize("m", [1, 2])
def test_layers_agree(m, K, boundary, prec):
    print(f"[layered] m={m} K={K} {boundary} {prec}", file=sys.stderr, flush=True)
    nodes = [k + (boundary == "walls") for k in K]
    assert (_layered_tiles(nodes) >= 512) == (K != (65, 9, 170))
    rng = np.random.default_rng(m + sum(K))
    plan = hl.Plan(3, m, K, cfl=0.5, precision=prec, boundary=boundary)
    ps, us = plan.host_shapes()
    P = rng.uniform(-1, 1, ps)
    P = inputs.zero_on_walls(P, 3) if boundary == "walls" else P
    p0, u0 = plan.alloc()
    plan.init(p0, u0, P, rng.uniform(-1, 1, us))
    got = []
    for tile in ((0, 0), (128, 2)):
        plan.set_tile(*tile)
        p, u = p0.clone(), u0.clone()
        plan.p_half(p, u)
        pb, ub = p0.clone(), u0.clone()
        plan.adjoint_step(pb, ub, 1)
        got.append((p, pb, ub))
    torch.cuda.synchronize()
    assert not torch.equal(got[0][0], p0)
    for a, b in zip(*got):
        assert torch.equal(a, b)
