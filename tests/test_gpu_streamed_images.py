"""The bf16 filter gradient over images whose operands stream into LDS, against the CPU oracle at the sizes where it can go wrong.

Bounds as in test_gpu_bf16_any_channels.py: the rounding of fp32 sums."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, force, owt  # noqa: E402
from test_gpu_bf16_any_channels import check, tensors  # noqa: E402

# N, C, H, W, K, R, S, pad: one image group less or more than full, channels and filters less and more than a tile, one row, rows of
# one output, no padding, padding on one side of the filter only, padding as wide as the filter, more filter rows than image rows
ROWS = {3: [(17, 40, 9, 7, 136, 3, 3, 1), (33, 136, 5, 9, 264, 3, 3, 1), (16, 200, 4, 4, 8, 3, 3, 1), (3, 8, 6, 11, 8, 5, 3, (2, 1)), (2, 32, 3, 3, 64, 3, 3, 0),
            (1, 264, 1, 6, 16, 1, 3, (0, 1)), (15, 8, 6, 5, 24, 3, 3, (1, 0)), (5, 16, 4, 3, 8, 3, 3, (1, 2))],
        5: [(18, 72, 11, 6, 200, 5, 5, 2), (1, 64, 6, 8, 64, 3, 5, (1, 2)), (15, 8, 5, 5, 8, 5, 5, 0), (4, 40, 9, 5, 16, 1, 5, (0, 2)), (33, 24, 2, 13, 72, 3, 5, (1, 1))]}


@pytest.mark.parametrize("variant,S", [(0, 3), (1, 3), (2, 3), (3, 3), (4, 5), (5, 5), (6, 5)])
@pytest.mark.parametrize("split", [0, 1, 4])
def test_filter_gradient_with_streamed_operands(variant, S, split):
    m = owt()
    for i, shape in enumerate(ROWS[S]):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 1, 1700 + i)
        for alpha, beta in ((1.0, 0.0), (0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, False)
            if case.P > H:
                continue                                         # (more output rows than input rows: the gather kernel's)
            dw0, db0 = np.full(case.shape_w, 2.0, np.float32), np.full((K,), 3.0, np.float32)
            with force(100 + variant, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                print("case", shape, plan)
                sys.stdout.flush()
                assert plan.startswith("ifilter16b"), plan
                dw, db = case.bwd_filter(x, dy, None, alpha, beta, dw0, db0)
            rw, rb = oracle.conv_bwd_filter(x, dy, (R, S), 1, pad, alpha=alpha, beta=beta, dw=dw0, db=db0)
            sw, sb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), 1, pad)
            L = N * case.P * case.Q
            check(dw, rw, sw + 2.0, L, "dw")
            check(db, rb, sb + 3.0, L, "dbias")


def test_infinities_stay_with_the_taps_that_meet_them():
    # an infinite value of x at either end of a row: the taps that never meet it keep what they are without it, although the row's
    # neighbour in memory is the next row's first column
    shape = N, C, H, W, K, R, S, pad = (5, 40, 4, 6, 32, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 1, 1790)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, False)
    for at in ((0, 0, 0), (0, 1, W - 1), (4, H - 1, 0)):
        xi = x.copy()
        xi[at + (7,)] = np.inf
        ref, _ = oracle.conv_bwd_filter(xi, dy, (R, S), 1, pad)
        clean, _ = oracle.conv_bwd_filter(x, dy, (R, S), 1, pad)
        met = ~np.isfinite(ref)
        assert met.any() and not met.all()
        for variant in range(4):
            with force(100 + variant, 1):
                dw, _ = case.bwd_filter(xi, dy, None)
            print("case", at, variant)
            sys.stdout.flush()
            assert (np.isfinite(dw) == ~met).all()
            assert np.allclose(dw[~met], clean[~met], rtol=1e-4, atol=1e-4)
