"""Tuning goes by time, also where the untuned choice weighs a kernel by more than that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import empty, owt, to_dev, workspace  # noqa: E402


# one and two images, which leave 14 or 15 in 16 of the kernels over images zeros: the gather kernel takes 0.6 to 0.7 of their time
@pytest.mark.parametrize("shape", [(2, 44, 7, 274, 256, 3, False), (1, 18, 42, 346, 32, 5, True), (2, 14, 53, 335, 480, 3, True), (1, 11, 52, 96, 78, 5, False)])
def test_fp32_filter_gradients_of_one_or_two_images_are_timed_gathering(shape):
    m = owt()
    N, H, W, C, K, R, masked = shape
    g = np.random.default_rng(3200)
    x, dy, y = (to_dev(g.standard_normal(s, dtype=np.float32)) for s in ((N, H, W, C), (N, H, W, K), (N, H, W, K)))
    w, dw, db = empty((K, R, R, C)), empty((K, R, R, C)), empty((K,))
    d = m.conv_desc(N, C, H, W, K, R, R, 1, R // 2, m.OWT_F32, m.OWT_BIAS | (m.OWT_RELU if masked else 0))
    assert m.owt_conv_plan_describe(d, 2).startswith(("xfilter", "xgather"))
    m.owt_conv_autotune(d, 2, x, w, None, y, dy, None, dw, db, workspace(m.owt_conv_workspace_bytes(d, 2)))
    assert m.owt_conv_plan_describe(d, 2).startswith("igemm"), m.owt_conv_plan_describe(d, 2)
