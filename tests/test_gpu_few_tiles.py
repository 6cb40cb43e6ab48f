"""The split-operand convolution kernel for layers of few tiles (groups of wavefronts share a work-group's taps), against the CPU
oracle and 64 bits, with the bounds of test_gpu_split.py."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, empty, force, owt, to_dev, to_host, workspace  # noqa: E402
from test_gpu_split import ENDS, check, check_ends, conv64, tensors  # noqa: E402

# N, C, H, W, K, R, S, pad: one pixel tile less or more than full, channel counts with a short last chunk (a multiple of four and
# not), ragged column tiles, taps that the groups share evenly and not, one chunk, no padding, rows that need each of the panels
SHAPES = [(4, 40, 13, 13, 136, 3, 3, 1), (3, 64, 9, 27, 71, 5, 5, 2), (2, 37, 9, 14, 12, 3, 5, (1, 2)), (1, 3, 5, 5, 4, 3, 3, 1), (5, 50, 6, 7, 66, 3, 3, 1),
          (1, 16, 7, 45, 33, 5, 5, 2), (2, 9, 4, 50, 32, 3, 3, 1), (1, 5, 3, 4, 2, 2, 4, (0, 0))]


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("split", [1, 2, 3])
def test_convolution_kernel_of_few_tiles(variant, split):
    m = owt()
    ran = 0
    for i, shape in enumerate(SHAPES):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 1500 + i)
        for relu in (False, True):
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, relu)
            with force(44 + variant, split):
                plans = [m.owt_conv_plan_describe(case.desc, p) for p in (0, 1)]
                print("case", shape, "relu", relu, plans)
                sys.stdout.flush()
                if plans[0].startswith("xconvs"):
                    size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), 1, pad, False)
                    check(case.fwd(x, w, b), oracle.conv_fwd(x, w, b, 1, pad, relu), size, R * S * C, "y")
                    ran += 1
                if plans[1].startswith("xconvs"):
                    size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad, y=y if relu else None)
                    check(case.bwd_data(dy, y, w), oracle.conv_bwd_data(dy, w, (H, W), 1, pad, y=y if relu else None), size, R * S * K, "dx")
                    ran += 1
    assert ran >= 2 * (2 * len(SHAPES) - 5)              # (a few tiles' rows fit no panel; unpadded backward-data has no panel)


def test_few_tiles_with_the_mask_of_the_layer_below():
    m = owt()
    N, C, H, W, K, R, S, pad = shape = (4, 40, 13, 13, 136, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 1530)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, False)
    size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad)
    for variant in (0, 1, 2):
        for split in (1, 3):
            with force(44 + variant, split):
                dx = empty(case.shape_x)
                m.owt_conv_bwd_data_relu_in(case.desc, to_dev(dy), None, to_dev(w), to_dev(x), dx, case.ws(1))
                torch.cuda.synchronize()
            check(to_host(dx), oracle.conv_bwd_data(dy, w, (H, W), 1, pad) * (x > 0), size, R * S * K, "dx masked by x > 0")


def test_few_tiles_keep_infinities_and_nans():
    N, C, H, W, K, R, S, pad = shape = (1, 24, 9, 9, 40, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 1540)
    x[0, 1, 1, 3], x[0, 1, 6, 9], x[0, 6, 1, 20], x[0, 6, 6, 0] = np.inf, -np.inf, np.nan, np.float32(3.4e38)
    x[0, 8, 8, 5] = np.float32(-3.4028234e38)
    w[:, :, :, 0] *= np.float32(0.01)
    with np.errstate(all="ignore"):
        want = np.zeros((H, W, K))
        xp = np.zeros((H + 2, W + 2, C)); xp[1:-1, 1:-1] = x[0]
        for r in range(R):
            for s in range(S):
                want += xp[r:r + H, s:s + W] @ w[:, r, s].astype(np.float64).T
        want = want.astype(np.float32)
    for variant in (0, 1, 2):
        with force(44 + variant, 1):
            got = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", False, False).fwd(x, w, None)[0]
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
        fine = np.isfinite(want)
        assert fine.any() and np.max(np.abs(got[fine] - want[fine]) / (np.abs(want[fine]) + 1e-4 * np.median(np.abs(want[fine])))) < 1e-3
    # an infinite filter value in the first channel of a tap, next to the last channels of the tap before it
    w2 = tensors((1, 21, 9, 9, 40, 3, 3, 1), 1541)[1]
    w2[7, 1, 1, 0] = np.inf
    x2 = np.zeros((1, H, W, 21), np.float32)
    x2[0, 4, 4, 5] = 1.0
    with force(46, 1):
        got = ConvCase(1, 21, H, W, K, R, S, 1, pad, "f32", False, False).fwd(x2, w2, None)[0]
    assert np.isfinite(got[:, :, :7]).all() and np.isfinite(got[:, :, 8:]).all() and np.isnan(got[3:6, 3:6, 7]).sum() >= 1


@pytest.mark.parametrize("a,b", ENDS)
def test_few_tiles_at_the_ends_of_the_range(a, b):
    m = owt()
    with np.errstate(under="ignore"):
        N, C, H, W, K, R, S, stride, pad = (2, 24, 9, 10, 40, 3, 3, 1, 1)
        g = np.random.default_rng(1550)
        case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)
        x = (g.standard_normal(case.shape_x) * a).astype(np.float32)
        w = (g.standard_normal(case.shape_w) * b).astype(np.float32)
        dy = (g.standard_normal(case.shape_y) * a).astype(np.float32)
        y = g.standard_normal(case.shape_y).astype(np.float32)
        masked = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, True)
        ref = conv64(x, w, stride, pad, case.P, case.Q)[0]
        back = conv64(dy * (y > 0), w[:, ::-1, ::-1].transpose(3, 1, 2, 0), 1, pad, H, W)[0]
        for variant in (0, 1, 2):
            for split in (1, 2):
                with force(44 + variant, split):
                    assert m.owt_conv_plan_describe(case.desc, 0).startswith("xconvs")
                    check_ends(case.fwd(x, w, None), ref, R * S * C, "y")
                    check_ends(masked.bwd_data(dy, y, w), back, R * S * K, "dx")


def test_few_tiles_leave_a_product_just_below_the_largest_number_finite():
    one, big = np.float32(float.fromhex("0x1.ffp0")), np.float32(float.fromhex("0x1.ffp126"))
    case = ConvCase(1, 20, 5, 6, 9, 3, 3, 1, 1, "f32", False, False)
    for u, v in ((one, big), (big, one), (-one, big)):
        x, w = np.zeros(case.shape_x, np.float32), np.zeros(case.shape_w, np.float32)
        x[0, 2, 2, 2], w[4, 1, 1, 2] = u, v
        ref = conv64(x, w, 1, 1, case.P, case.Q)[0].astype(np.float32)
        assert np.isfinite(ref).all()
        for variant in (0, 1, 2):
            with force(44 + variant, 1):
                assert np.array_equal(case.fwd(x, w, None), ref)


# Layers that the planner gives to this kernel and gave to `splits` splits of the other: N, C, H, W, K, R, S, pad, pass, splits.
# Bound: a rounding of the sum of i of n equal random products counts i/n, so the second layer's 72 instructions count 5 in eight
# chains of nine and 3 in adding those up; here 6 in chains of 12, 10 and 6 and 2 in adding them up, against 10 and 2 in four chains
# of 24 and 16.  Ratios of the roots: 1.02 here, 1.23 with four chains; 1.1 lies between, and the errors are averages over thousands of
# outputs whose ratio moves by 1 % from one set of inputs to the next.
@pytest.mark.parametrize("shape,p,splits", [((5, 224, 20, 12, 383, 3, 3, 1), 0, 7), ((12, 128, 26, 35, 19, 3, 3, 1), 0, 8), ((4, 384, 33, 7, 96, 3, 3, 1), 1, 6)])
def test_few_tiles_are_no_further_from_64_bits_than_many_splits(shape, p, splits):
    m = owt()
    N, C, H, W, K, R, S, pad = shape
    g = np.random.default_rng(1560)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", False, False)
    x = np.maximum(g.standard_normal(case.shape_x, dtype=np.float32), 0)
    w = g.standard_normal(case.shape_w, dtype=np.float32) * np.float32(0.01)
    dy = g.standard_normal(case.shape_y, dtype=np.float32)
    ref = conv64(x, w, 1, pad, H, W)[0] if p == 0 else conv64(dy, w[:, ::-1, ::-1].transpose(3, 1, 2, 0), 1, pad, H, W)[0]
    off = []
    for tile, split, name in ((43, splits, "xconv "), (-1, 0, "xconvs ")):
        with force(tile, split):
            assert m.owt_conv_plan_describe(case.desc, p).startswith(name), m.owt_conv_plan_describe(case.desc, p)
            got = case.fwd(x, w, None) if p == 0 else case.bwd_data(dy, None, w)
        off.append(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(shape, off)
    assert off[1] <= 1.1 * off[0]


def test_the_default_choice_runs_it_where_tiles_are_few_and_not_elsewhere():
    m = owt()
    plan = lambda s, p: m.owt_conv_plan_describe(m.conv_desc(*s[:7], 1, s[7], m.OWT_F32, m.OWT_BIAS), p)
    for p in (0, 1):
        assert plan((8, 3, 32, 32, 16, 5, 5, 2), p).startswith("xconvs")
        assert plan((2, 19, 19, 7, 160, 3, 3, 1), p).startswith("xconvs")
        assert plan((128, 192, 13, 13, 384, 3, 3, 1), p).startswith("xconv ")
        assert plan((128, 64, 27, 27, 192, 5, 5, 2), p).startswith("xconv ")


# panels of two and three chunks: whole ones, a short last one of either length, a single short one, channels that end inside a chunk,
# a panel whose taps the groups share evenly and not (N, C, H, W, K, R, S, pad; the smallest panel of each tile)
@pytest.mark.parametrize("variant,chunks", [(0, 3), (1, 2), (2, 2)])
@pytest.mark.parametrize("split", [1, 2])
def test_panels_of_several_chunks(variant, chunks, split):
    m = owt()
    for i, (C, K) in enumerate([(16 * c - cut, 16 * (chunks + 1) - 5) for c in range(1, 2 * chunks + 2) for cut in (0, 3)]):
        for R, S, pad in ((3, 3, 1), (2, 4, (1, 2))):
            shape = N, _, H, W = (3, C, 7, 8)
            shape += (K, R, S, pad)
            x, w, b, dy, y = tensors(shape, 1580 + i)
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, True)
            with force(44 + variant, split):
                plans = [m.owt_conv_plan_describe(case.desc, p) for p in (0, 1)]
                print("case", shape, plans)
                sys.stdout.flush()
                if plans[0].startswith("xconvs"):                # (eight groups want eight taps)
                    size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), 1, pad, False)
                    check(case.fwd(x, w, b), oracle.conv_fwd(x, w, b, 1, pad, True), size, R * S * C, "y")
                if plans[1].startswith("xconvs"):
                    size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad, y=y)
                    check(case.bwd_data(dy, y, w), oracle.conv_bwd_data(dy, w, (H, W), 1, pad, y=y), size, R * S * K, "dx")
            assert any(p.startswith("xconvs") for p in plans), plans
