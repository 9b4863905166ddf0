"""3D grids of very many layers of a few nodes: from m = 2 on a 64 x 4 tile has 512
work-items, and 2^23 layers of one tile would be a launch of 2^32 work-items.  Such
plans start with a smaller tile.  The grid repeats a small one along z with its
spacing and dt, so every copy must equal the small grid's result bit for bit."""

import sys

import numpy as np
import pytest

from paper_1808_10481_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


def test_more_layers_than_a_launch_of_default_tiles():
    copies, K, m = 940000, (2, 2, 9), 2
    print(f"[layers] m={m} {K} x{copies}", file=sys.stderr, flush=True)
    big = K[:2] + (K[2] * copies,)
    assert big[2] > 1 << 23
    small = hl.Plan(3, m, K, length=[float(k) for k in K], dt=0.4, precision="fp32")
    large = hl.Plan(3, m, big, length=[float(k) for k in big], dt=0.4, precision="fp32")
    assert tuple(small.info.tile) == (64, 4)
    tx, ty = large.info.tile
    assert -(-K[0] // tx) * -(-K[1] // ty) * big[2] * 2 * -(-tx * ty // 64) * 64 < 1 << 32
    rng = np.random.default_rng(3)
    p, u = small.alloc()
    small.init(p, u, inputs.random_data(rng, 3, m, K), inputs.random_data(rng, 3, m, K, ncomp=3))

    def repeated(x, fields):
        return x.view(fields, 1, -1).expand(-1, copies, -1).reshape(-1)

    P, U = repeated(p, 27), repeated(u, 81)
    small.step(p, u, 1)
    large.step(P, U, 1)
    small.adjoint_step(p, u, 1)
    large.adjoint_step(P, U, 1)
    torch.cuda.synchronize()
    for big_field, field, n in ((P, p, 27), (U, u, 81)):
        planes = big_field.view(n, copies, -1)
        for c in range(n):
            assert bool((planes[c] == field.view(n, 1, -1)[c]).all()), c
