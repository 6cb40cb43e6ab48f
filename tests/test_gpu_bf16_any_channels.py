"""The bf16 kernels that take any channel counts, against the CPU oracle at the sizes where they can go wrong.

Bounds.  Products of bf16 values are exact in fp32, so what differs from the oracle is the rounding of fp32 sums: with
S = sum |a*b| of an output, (L/16 + 16) * 2^-24 * S for a reduction of length L, one rounding of S per 16-deep matrix
instruction plus one instruction's worth (in practice the roundings are independent and far smaller).  Outputs stored as
bf16 are rounded once more, by 2^-8 of the value at most."""
import re
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, empty, force, owt, to_dev, to_host, workspace  # noqa: E402


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


# N, C, H, W, K, R, S, stride, pad: rows of any length, less and more than a tile of filters and of places, filters odd and even,
# one tap, a stride along one side only, one position
ANY = [(5, 3, 51, 57, 33, 11, 11, 4, 2), (17, 3, 30, 31, 64, 7, 7, 4, 2), (16, 5, 19, 20, 70, 3, 3, 2, 1), (33, 37, 6, 5, 45, 1, 1, 1, 0), (2, 7, 23, 17, 5, 5, 4, (3, 1), (2, 1)), (1, 2, 7, 7, 3, 7, 7, 1, 0)]


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("split", [0, 1, 4])
def test_filter_gradient_of_any_geometry(variant, split):
    m = owt()
    for i, shape in enumerate(ANY):
        N, C, H, W, K, R, S, stride, pad = shape
        x, w, b, dy, y = tensors((N, C, H, W, K, R, S, pad), stride, 1220 + i)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "bf16", True, relu)
            dw0, db0 = np.full(case.shape_w, 2.0, np.float32), np.full((K,), 3.0, np.float32)
            with force(88 + variant, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                print("case", shape, "relu", relu, plan)
                sys.stdout.flush()
                assert plan.startswith(("sfilter16x", "igather16")), plan
                dw, db = case.bwd_filter(x, dy, y, alpha, beta, dw0, db0)
            mask = y if relu else None
            rw, rb = oracle.conv_bwd_filter(x, dy, (R, S), stride, pad, y=mask, alpha=alpha, beta=beta, dw=dw0, db=db0)
            sw, sb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), stride, pad, y=mask)
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


# N, C, H, W, K, R, S, pad: reduction channels odd, even and whole eights with a short last chunk or a single short one; result
# columns odd, even, more than a tile; a tile of pixels less or more than full; rows that need the largest panel
CONV = [(5, 37, 9, 7, 45, 3, 3, 1), (7, 70, 9, 11, 66, 3, 3, 1), (3, 33, 11, 6, 34, 5, 5, 2), (2, 1, 6, 7, 1, 3, 3, 1), (1, 31, 8, 55, 130, 5, 5, 2),
        (2, 72, 13, 9, 5, 3, 5, (1, 2)), (3, 10, 5, 40, 3, 5, 3, (2, 1)), (1, 97, 1, 3, 35, 1, 3, (0, 1))]


@pytest.mark.parametrize("split", [0, 1, 2])
@pytest.mark.parametrize("shape", CONV)
def test_convolution_of_any_channel_counts(shape, split):
    m = owt()
    N, C, H, W, K, R, S, pad = shape
    x, w, b, dy, y = tensors(shape, 1, 1300)
    for relu in (False, True):
        case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, relu)
        with force(90, split):
            plans = [m.owt_conv_plan_describe(case.desc, p) for p in (0, 1)]
            print("case", shape, "relu", relu, plans)
            sys.stdout.flush()
            assert all(p.startswith("dconv16x") for p in plans), plans
            got, dx = case.fwd(x, w, b), case.bwd_data(dy, y, w)
        size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), 1, pad, False)
        check(got, oracle.conv_fwd(x, w, b, 1, pad, relu), size, R * S * C, "y", 2.0 ** -8)
        size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad, y=y if relu else None)
        check(dx, oracle.conv_bwd_data(dy, w, (H, W), 1, pad, y=y if relu else None), size, R * S * K, "dx", 2.0 ** -8)


def test_convolution_of_any_channel_counts_with_the_mask_of_the_layer_below():
    m = owt()
    for shape in ((5, 37, 9, 7, 45, 3, 3, 1), (7, 70, 9, 11, 66, 3, 3, 1)):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 1, 1310)
        case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, False)
        for split in (1, 2):
            with force(90, split):
                dx = empty(case.shape_x, "bf16")
                m.owt_conv_bwd_data_relu_in(case.desc, to_dev(dy, "bf16"), None, to_dev(w, "bf16"), to_dev(x, "bf16"), dx, case.ws(1))
                torch.cuda.synchronize()
            size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad)
            check(to_host(dx), oracle.conv_bwd_data(dy, w, (H, W), 1, pad) * (x > 0), size, R * S * K, "dx masked by x > 0", 2.0 ** -8)


def test_channels_of_the_next_pixel_do_not_reach_a_short_chunk():
    # the last piece of a pixel's channels is loaded 16 bytes wide: what follows belongs to the next pixel and may be infinite
    m = owt()
    for shape in ((2, 37, 5, 6, 40, 3, 3, 1), (2, 38, 5, 6, 39, 3, 3, 1)):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 1, 1320)
        case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, False)
        x[1, 0, 0, :] = np.inf                                   # image 1's first pixel follows image 0's last
        dy[1, 0, 0, :] = np.inf
        with force(90):
            got, dx = case.fwd(x, w, b), case.bwd_data(dy, None, w)
        assert np.isfinite(got[0]).all() and np.isfinite(dx[0]).all()
        assert np.isfinite(got[1, 2:]).all() and np.isfinite(got[1, :, 2:]).all() and not np.isfinite(got[1, :2, :2]).any()
        assert np.isfinite(dx[1, 2:]).all() and np.isfinite(dx[1, :, 2:]).all() and not np.isfinite(dx[1, :2, :2]).any()


# N, C, H, W, K, R, S, stride, pad: rows of any length, one to three chunks of a block's values, one split in three
BLOCKS = [(3, 3, 51, 57, 33, 11, 11, 4, 2), (2, 3, 30, 31, 64, 7, 7, 4, 2), (2, 5, 19, 20, 70, 3, 3, 2, 1), (1, 7, 23, 17, 5, 5, 4, (3, 4), (2, 1)), (2, 1, 40, 9, 8, 6, 5, (4, 2), 0)]


@pytest.mark.parametrize("split", [0, 1, 3])
@pytest.mark.parametrize("shape", BLOCKS)
def test_strided_forward_over_blocks(shape, split):
    m = owt()
    N, C, H, W, K, R, S, stride, pad = shape
    x, w, b, dy, y = tensors((N, C, H, W, K, R, S, pad), stride, 1330)
    for relu in (False, True):
        case = ConvCase(N, C, H, W, K, R, S, stride, pad, "bf16", True, relu)
        with force(90, split):
            plan = m.owt_conv_plan_describe(case.desc, 0)
            print("case", shape, "relu", relu, plan)
            sys.stdout.flush()
            assert plan.startswith("sconv16x"), plan
            got = case.fwd(x, w, b)
        size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), stride, pad, False)
        check(got, oracle.conv_fwd(x, w, b, stride, pad, relu), size, R * S * C, "y", 2.0 ** -8)


@pytest.mark.parametrize("split", [1, 2])
def test_strided_forward_meets_no_value_outside_its_windows(split):
    # a 5 x 7 filter at stride 4 x 4: blocks hold pixels that a window does not
    N, C, H, W, K, R, S, stride, pad = 2, 3, 37, 41, 20, 5, 7, 4, 2
    x, w, b, dy, y = tensors((N, C, H, W, K, R, S, pad), stride, 1340)
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "bf16", True, False)
    with force(90, split):
        assert owt().owt_conv_plan_describe(case.desc, 0).startswith("sconv16x")
        clean = case.fwd(x, w, b)
        for value in (np.inf, -np.inf, np.nan):
            for n, h, c in ((0, 0, 0), (0, 19, 22), (1, H - 1, W - 1)):
                xi = x.copy()
                xi[n, h, c, 1] = value
                got = case.fwd(xi, w, b)
                for p in range(case.P):
                    for q in range(case.Q):
                        meets = 0 <= h - (p * 4 - 2) < R and 0 <= c - (q * 4 - 2) < S
                        assert not meets or not np.isfinite(got[n, p, q]).any()
                        assert meets or np.array_equal(got[n, p, q], clean[n, p, q])
                assert np.array_equal(got[1 - n], clean[1 - n])


def test_calls_with_the_scratch_of_the_gather_kernel_still_run():
    # the padded filters need workspace; a call that brings what the kernels before these asked for is served by those, to the bit
    m = owt()
    shape = N, C, H, W, K, R, S, pad = (40, 5, 9, 8, 6, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 1, 1350)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, False)
    dev = [to_dev(t, "bf16") for t in (x, w, dy)] + [to_dev(b)]
    calls = (lambda out, ws: m.owt_conv_fwd(case.desc, dev[0], dev[1], dev[3], out, ws),
             lambda out, ws: m.owt_conv_bwd_data(case.desc, dev[2], None, dev[1], out, ws),
             lambda out, ws: m.owt_conv_bwd_filter(case.desc, dev[0], dev[2], None, 1.0, 0.0, out, None, ws))
    for p, call in enumerate(calls):
        assert m.owt_conv_plan_describe(case.desc, p).startswith(("dconv16x", "dconv16s") if p < 2 else "ifilter16")
        out = [empty((case.shape_y, case.shape_x, case.shape_w)[p], "bf16" if p < 2 else "f32") for _ in range(2)]
        with force(flags=m.OWT_FORCE_NO_BF16_MFMA):
            assert m.owt_conv_plan_describe(case.desc, p).startswith("igemm")
            need = m.owt_conv_workspace_bytes(case.desc, p)
            assert p == 2 or need == 0
            call(out[0], workspace(need) if need else None)
        call(out[1], workspace(need) if need else None)
        torch.cuda.synchronize()
        if p < 2:
            assert torch.equal(out[0], out[1])
        else:
            assert (out[0] - out[1]).norm() <= 1e-5 * out[0].norm()


# filters, taps, channels whose product leaves 0 to 3 results past the last group of four, times few, some and many splits
@pytest.mark.parametrize("K,R,C", [(4, 3, 8), (5, 3, 5), (1, 3, 2), (7, 3, 13), (33, 1, 1), (3, 3, 9)])
@pytest.mark.parametrize("split", [2, 6, 7, 32, 33, 70])
def test_split_sums_of_any_length(K, R, C, split):
    m = owt()
    shape = (18, C, 7, 9, K, R, R, R // 2)
    x, w, b, dy, y = tensors(shape, 1, 1400)
    case = ConvCase(*shape[:7], 1, shape[7], "bf16", True, False)
    dw0, db0 = np.full(case.shape_w, 2.0, np.float32), np.full((K,), 3.0, np.float32)
    for tile in ((80, 83, 89) if R == 3 else (89,)):
        with force(tile, split):
            plan = m.owt_conv_plan_describe(case.desc, 2)
            print("case", K, R, C, plan)
            sys.stdout.flush()
            assert plan.startswith(("ifilter16", "igather16")) and "splitk1 " not in plan, plan
            dw, db = case.bwd_filter(x, dy, None, 0.5, -0.25, dw0, db0)
        rw, rb = oracle.conv_bwd_filter(x, dy, (R, R), 1, R // 2, alpha=0.5, beta=-0.25, dw=dw0, db=db0)
        sw, sb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, R), 1, R // 2)
        check(dw, rw, sw + 2.0, 18 * 63, "dw")
        check(db, rb, sb + 3.0, 18 * 63, "dbias")


def test_first_layers_of_either_kernel_go_to_the_faster_one():
    m = owt()
    plan = lambda N, H, K, R: m.owt_conv_plan_describe(m.conv_desc(N, 3, H, H, K, R, R, 4, 2, m.OWT_BF16, m.OWT_BIAS), 0)
    for layer in ((128, 224, 96, 11), (89, 204, 96, 11), (391, 204, 32, 7), (5, 204, 32, 11), (10, 80, 64, 7)):
        text = plan(*layer)
        a, b = re.search(r"grid(\d+)x(\d+)", text).groups()
        assert text.startswith("sconv16 ") and int(a) * int(b) <= 256, text
    for layer in ((349, 187, 64, 11), (490, 95, 32, 11), (257, 52, 96, 11)):   # rows that sconv16 cannot take, and maps it leaves mostly idle
        assert plan(*layer).startswith("sconv16x"), plan(*layer)


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("split", [1, 2])
def test_convolution_of_few_tiles(variant, split):
    m = owt()
    ran = 0
    for shape in CONV + [(4, 64, 13, 13, 136, 3, 3, 1), (1, 16, 7, 45, 33, 5, 5, 2), (3, 40, 6, 7, 24, 3, 3, 1)]:
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 1, 1350)
        for relu in (False, True):
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "bf16", True, relu)
            with force(92 + variant, split):
                plans = [m.owt_conv_plan_describe(case.desc, p) for p in (0, 1)]
                print("case", shape, "relu", relu, plans)
                sys.stdout.flush()
                if plans[0].startswith("dconv16s"):
                    size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), 1, pad, False)
                    check(case.fwd(x, w, b), oracle.conv_fwd(x, w, b, 1, pad, relu), size, R * S * C, "y", 2.0 ** -8)
                    ran += 1
                if plans[1].startswith("dconv16s"):
                    size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad, y=y if relu else None)
                    check(case.bwd_data(dy, y, w), oracle.conv_bwd_data(dy, w, (H, W), 1, pad, y=y if relu else None), size, R * S * K, "dx", 2.0 ** -8)
                    ran += 1
            if not relu and plans[1].startswith("dconv16s"):
                with force(92 + variant, split):
                    dx = empty(case.shape_x, "bf16")
                    m.owt_conv_bwd_data_relu_in(case.desc, to_dev(dy, "bf16"), None, to_dev(w, "bf16"), to_dev(x, "bf16"), dx, case.ws(1))
                    torch.cuda.synchronize()
                size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad)
                check(to_host(dx), oracle.conv_bwd_data(dy, w, (H, W), 1, pad) * (x > 0), size, R * S * K, "dx masked by x > 0", 2.0 ** -8)
    assert ran >= 4 * 9                                  # (all but the one of three taps and one whose rows fit no panel)


def test_few_tiles_meet_no_channel_of_the_next_pixel_or_tap():
    m = owt()
    for C in (5, 18, 33):                                # loads of one and of two values, one short chunk and a second one
        shape = (2, C, 6, 7, 9, 3, 3, 1)
        x, w, _, dy, y = tensors(shape, 1, 1360)
        x[0, 2, 3, 0] = np.inf
        w[4, 1, 1, 0] = np.nan
        ref = np.zeros((2, 6, 7, 9))
        xp = np.zeros((2, 8, 9, C)); xp[:, 1:-1, 1:-1] = x
        with np.errstate(invalid="ignore"):
            for r in range(3):
                for s in range(3):
                    ref += xp[:, r:r + 6, s:s + 7] @ w[:, r, s].astype(np.float64).T
        for variant in (0, 1, 2):
            with force(92 + variant, 1):
                case = ConvCase(2, C, 6, 7, 9, 3, 3, 1, 1, "bf16", False, False)
                assert m.owt_conv_plan_describe(case.desc, 0).startswith("dconv16s")
                got = case.fwd(x, w, None)
            assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
            assert np.array_equal(np.isneginf(got), np.isneginf(ref)) and np.isfinite(got).any()


def test_small_bf16_layers_go_to_the_kernel_of_few_tiles_and_large_ones_do_not():
    m = owt()
    plan = lambda s, p: m.owt_conv_plan_describe(m.conv_desc(*s[:7], 1, s[7], m.OWT_BF16, m.OWT_BIAS), p)
    for p in (0, 1):
        for shape in ((3, 162, 7, 19, 43, 3, 3, 1), (2, 65, 17, 16, 31, 3, 3, 1), (1, 32, 15, 49, 32, 5, 5, 2)):
            assert plan(shape, p).startswith("dconv16s"), plan(shape, p)
        for shape in ((2, 64, 17, 16, 32, 3, 3, 1), (128, 192, 13, 13, 384, 3, 3, 1), (128, 64, 27, 27, 192, 5, 5, 2), (405, 57, 38, 26, 32, 3, 3, 1)):
            assert not plan(shape, p).startswith("dconv16s"), plan(shape, p)
