"""The y-group of 3D plans: hl_plan_info reports what the half-steps run, an
explicit value (hl_set_tile) is used as given, and 0 is the default: 4, or 2
with variable kappa and at m = 0."""

import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1808_10481_amd import hl  # noqa: E402


@pytest.mark.parametrize("m", [1, 2])
def test_reported_y_group(m):
    print(f"[ygroup] m={m}", file=sys.stderr, flush=True)
    K = (5, 37, 3)  # ten tile rows
    plan = hl.Plan(3, m, K)
    assert plan.info.ygroup == 4
    for given, used in ((1, 1), (3, 3), (8, 8), (40, 10), (0, 4)):
        plan.set_tile(64, 4, given)
        assert plan.info.ygroup == used
    kp, ku = (np.zeros(K + (2 * m + 2,) * 3) for _ in range(2))
    kp[..., 0, 0, 0] = ku[..., 0, 0, 0] = 1.0
    plan.set_kappa(kp, ku)
    for given, used in ((0, 2), (1, 1), (5, 5)):
        plan.set_tile(64, 4, given)
        assert plan.info.ygroup == used
    plan.set_kappa(None, None)
    plan.set_tile()
    assert plan.info.ygroup == 4


def test_default_at_m0():
    print("[ygroup] m=0", file=sys.stderr, flush=True)
    plan = hl.Plan(3, 0, (5, 37, 3))
    for given, used in ((0, 2), (1, 1), (4, 4)):
        plan.set_tile(64, 4, given)
        assert plan.info.ygroup == used
