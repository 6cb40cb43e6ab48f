"""The bf16 kernels that take any channel counts, against the CPU oracle at the sizes where they can go wrong.

Bounds.  Products of bf16 values are exact in fp32, so what differs from the oracle is the rounding of fp32 sums: with
S = sum |a*b| of an output, (L/16 + 16) * 2^-24 * S for a reduction of length L, one rounding of S per 16-deep matrix
instruction plus one instruction's worth (in practice the roundings are independent and far smaller).  Outputs stored as
bf16 are rounded once more, by 2^-8 of the value at most."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, force, owt  # noqa: E402


def check(got, ref, size, L, what, stored=0.0):
    got, ref = got.astype(np.float64), ref.astype(np.float64)
    worst = np.max(np.abs(got - ref) / ((L / 16 + 16) * 2.0 ** -24 * size + stored * np.abs(ref) + 1e-30))
    print("  %s: %.3f of the bound" % (what, worst))
    sys.stdout.flush()
    assert worst <= 1.0, what


def tensors(shape, stride, seed):
    case = ConvCase(*shape[:7], stride, shape[7], "bf16", True, False)
    g = np.random.default_rng(seed)
    r = lambda s, scale=1.0: oracle.round_bf16(g.standard_normal(s, dtype=np.float32) * np.float32(scale))
    return (r(case.shape_x), r(case.shape_w, 0.05), g.standard_normal((shape[4],), dtype=np.float32), r(case.shape_y), r(case.shape_y))


# N, C, H, W, K, R, S, pad: one image group less or more than full, channels and filters odd, even and in whole blocks (loads of
# one or two channels), one row, no padding, padding on one side of the filter only, one channel
ROWS = {3: [(17, 37, 9, 7, 45, 3, 3, 1), (33, 70, 7, 9, 66, 3, 3, 1), (16, 64, 5, 4, 128, 3, 3, 1), (3, 1, 6, 11, 1, 5, 3, (2, 1)), (2, 34, 3, 3, 65, 3, 3, 0)],
        5: [(18, 33, 11, 6, 35, 5, 5, 2), (1, 72, 6, 8, 68, 3, 5, (1, 2)), (15, 64, 5, 5, 64, 5, 5, 0), (4, 2, 9, 5, 3, 1, 5, (0, 2))]}


@pytest.mark.parametrize("variant,S", [(0, 3), (1, 3), (2, 3), (3, 3), (4, 5), (5, 5), (6, 5)])
@pytest.mark.parametrize("split", [0, 1, 4])
def test_filter_gradient_with_the_reduction_over_images(variant, S, split):
    m = owt()
    for i, shape in enumerate(ROWS[S]):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 1, 1200 + i)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, relu)
            dw0, db0 = np.full(case.shape_w, 2.0, np.float32), np.full((K,), 3.0, np.float32)
            with force(80 + variant, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                print("case", shape, "relu", relu, plan)
                sys.stdout.flush()
                assert plan.startswith("ifilter16"), plan
                dw, db = case.bwd_filter(x, dy, y, alpha, beta, dw0, db0)
            mask = y if relu else None
            rw, rb = oracle.conv_bwd_filter(x, dy, (R, S), 1, pad, y=mask, alpha=alpha, beta=beta, dw=dw0, db=db0)
            sw, sb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), 1, pad, y=mask)
            L = N * case.P * case.Q
            check(dw, rw, sw + 2.0, L, "dw")
            check(db, rb, sb + 3.0, L, "dbias")


def test_filter_gradient_over_images_keeps_infinities_to_the_taps_that_meet_them():
    # an infinite value of x at the last column of a row: taps left of it never meet it, although its column is the first
    # row's neighbour in memory and still in the wavefront's ring when the next row starts
    m = owt()
    shape = N, C, H, W, K, R, S, pad = (5, 33, 4, 6, 34, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 1, 1290)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, False)
    for at in ((0, 0, 0), (0, 1, W - 1), (4, H - 1, 0)):
        xi = x.copy()
        xi[at + (7,)] = np.inf
        ref = case_dw(xi, dy, R, S, pad)
        for variant in range(4):
            for split in (0, 1):
                with force(80 + variant, split):
                    dw, _ = case.bwd_filter(xi, dy, None)
                print("case", at, variant, split)
                assert np.array_equal(np.isfinite(dw), np.isfinite(ref)) and np.array_equal(np.isnan(dw), np.isnan(ref))


def case_dw(x, dy, R, S, pad):
    """dw of dense tensors with non-finite values, tap by tap: only positions whose input pixel exists take part."""
    N, H, W, C = x.shape
    P, Q, K = dy.shape[1:]
    dw = np.zeros((K, R, S, C))
    with np.errstate(invalid="ignore"):
        for r in range(R):
            for s in range(S):
                p = [i for i in range(P) if 0 <= i + r - pad < H]
                q = [i for i in range(Q) if 0 <= i + s - pad < W]
                xs = x[:, [i + r - pad for i in p]][:, :, [i + s - pad for i in q]].reshape(-1, C).astype(np.float64)
                dw[:, r, s] = dy[:, p][:, :, q].reshape(-1, K).astype(np.float64).T @ xs
    return dw
