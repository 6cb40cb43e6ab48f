"""The last sum of a bias gradient, over the partial sums of a split reduction.

One partial sum is 1 and every other one just below half the spacing of fp32 above 1, so each addition to the first one is lost, and
the result shows how many of them one chain holds.  The bound is that of 256 chains added up in eight levels: (splits / 256 - 1 + 8)
roundings of at most 2^-24 of a sum below 2."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, force, owt  # noqa: E402


@pytest.mark.parametrize("dt,tile", [("f32", 61), ("bf16", 89)])
@pytest.mark.parametrize("H,W", [(32, 32), (32, 64), (64, 128)])
def test_bias_gradient_of_many_splits(dt, tile, H, W):
    splits, tiny = H * W, np.float32(255 * 2.0 ** -32)
    case = ConvCase(1, 1, H, W, 3, 1, 1, 1, 0, dt, True, False)
    x = np.zeros(case.shape_x, np.float32)
    with force(tile, splits):
        plan = owt().owt_conv_plan_describe(case.desc, 2)
        assert "gather" in plan and " splitk%d " % splits in plan, plan
        for first in (0, 5, splits - 1):
            dy = np.full(case.shape_y, tiny, np.float32)
            dy.reshape(splits, 3)[first] = 1.0
            got = case.bwd_filter(x, dy, None)[1].astype(np.float64)
            off = np.abs(got - (1.0 + (splits - 1) * float(tiny)))
            print(plan, first, off.max() * 2.0 ** 24)
            assert (off <= (splits / 256 - 1 + 8) * 2.0 ** -24).all(), (first, off)
