"""The kernels that multiply fp32 operands on the bf16 matrix unit, each operand split into three bf16 values, against
the CPU oracle at the sizes where they can go wrong.

Elementwise bound.  With S = sum |a*b| of an output (the oracle on absolute values): a 16-deep matrix instruction adds
exact products to an fp32 accumulator and rounds; whatever order it adds in, an error of 16 ulp of the largest partial
sum, 16 * 2^-24 S, per instruction is far more than it can make, and in practice the instructions of a reduction of
length L round independently.  The products left out are at most 2^-25 S in all.  Taken here: (L/16 + 16) * 2^-24 * S,
one rounding of S per instruction plus one instruction's worth.
2-norm bound.  Independent roundings of half an ulp give sqrt(L/16) * 0.29 * 2^-23 relative; 2^-23 * sqrt(L/16 + 4) is
taken.  Leaving out any of the six products taken would show 2^-17 or more.  It holds for a tensor of many values; a
bias gradient may be one value that cancels, so it gets the elementwise bound alone."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, empty, force, owt, to_dev, to_host, workspace  # noqa: E402


def check(got, ref, size, L, what, norm_too=True):
    got, ref = got.astype(np.float64), ref.astype(np.float64)
    worst = np.max(np.abs(got - ref) / ((L / 16 + 16) * 2.0 ** -24 * size + 1e-30))
    norm = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("  %s: %.3f of the elementwise bound, relative 2-norm error %.2e of %.2e" % (what, worst, norm, 2.0 ** -23 * np.sqrt(L / 16 + 4)))
    sys.stdout.flush()
    assert worst <= 1.0, what
    assert not norm_too or norm <= 2.0 ** -23 * np.sqrt(L / 16 + 4), what


def tensors(shape, seed, scale=1.0):
    N, C, H, W, K, R, S = shape[:7]
    g = np.random.default_rng(seed)
    case = ConvCase(*shape[:7], 1, shape[7], "f32", True, False)
    x = g.standard_normal(case.shape_x, dtype=np.float32) * np.float32(scale)
    w = g.standard_normal(case.shape_w, dtype=np.float32) * np.float32(0.05)
    b = g.standard_normal((K,), dtype=np.float32) * np.float32(scale)
    dy = g.standard_normal(case.shape_y, dtype=np.float32)
    y = g.standard_normal(case.shape_y, dtype=np.float32)
    return x, w, b, dy, y


# N, C, H, W, K, R, S, pad: one pixel tile less or more than full, channel counts with a short last chunk (a multiple of
# four and not), ragged column tiles, one tap, one chunk of many taps, maps narrower than a 32-pixel block
SHAPES = [(4, 40, 13, 13, 136, 3, 3, 1), (1, 16, 16, 16, 64, 1, 1, 0), (3, 64, 27, 27, 71, 5, 5, 2), (2, 37, 9, 14, 12, 3, 5, (1, 2)),
          (1, 3, 5, 5, 4, 3, 3, 1), (5, 50, 6, 7, 66, 3, 3, 0)]


@pytest.mark.parametrize("variant,split", [(0, 1), (1, 1), (2, 1), (3, 1), (0, 3), (1, 2), (2, 7), (3, 2)])
def test_split_convolution_kernel(variant, split):
    m = owt()
    for i, shape in enumerate(SHAPES):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 900 + i)
        for relu in (False, True):
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, relu)
            with force(40 + variant, split):
                plans = [m.owt_conv_plan_describe(case.desc, ps) for ps in (0, 1)]
                print("case", shape, "relu", relu, plans)
                sys.stdout.flush()
                same = all(2 * p == r - 1 for p, r in zip((pad, pad) if isinstance(pad, int) else pad, (R, S)))
                assert plans[0].startswith("xconv"), plans[0]
                assert plans[1].startswith("xconv") or not same, plans[1]
                got = case.fwd(x, w, b)
                dx = case.bwd_data(dy, y, w)
            size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), 1, pad, False)
            check(got, oracle.conv_fwd(x, w, b, 1, pad, relu), size, R * S * C, "y")
            size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad, y=y if relu else None)
            check(dx, oracle.conv_bwd_data(dy, w, (H, W), 1, pad, y=y if relu else None), size, R * S * K, "dx")


def test_split_convolution_with_the_mask_of_the_layer_below():
    m = owt()
    N, C, H, W, K, R, S, pad = shape = (4, 40, 13, 13, 136, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 930)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, False)
    ref = oracle.conv_bwd_data(dy, w, (H, W), 1, pad) * (x > 0)
    size = oracle.conv_bwd_data(np.abs(dy), np.abs(w), (H, W), 1, pad)
    for split in (1, 3):
        for variant in (0, 1, 3):
            with force(40 + variant, split):
                dx = empty(case.shape_x)
                m.owt_conv_bwd_data_relu_in(case.desc, to_dev(dy), None, to_dev(w), to_dev(x), dx, case.ws(1))
                torch.cuda.synchronize()
            check(to_host(dx), ref, size, R * S * K, "dx masked by x > 0")


# N, C, K of 1x1 maps, where backward-data is a plain matrix product: less than a tile, ragged, more than a tile
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("tile", [-1, 70])
@pytest.mark.parametrize("N,C,K", [(1, 1, 1), (37, 100, 72), (128, 256, 256), (70, 132, 20)])
def test_mask_of_the_layer_below_on_maps_of_one_pixel(dt, tile, N, C, K):
    m = owt()
    rnd = oracle.round_bf16 if dt == "bf16" else (lambda a: a)
    g = np.random.default_rng(935)
    x, dy, y = (rnd(g.standard_normal(s, dtype=np.float32)) for s in ((N, 1, 1, C), (N, 1, 1, K), (N, 1, 1, K)))
    w = rnd(g.standard_normal((K, 1, 1, C), dtype=np.float32))
    x[0, 0, 0, 0] = -1.0
    for relu in (False, True):
        case = ConvCase(N, C, 1, 1, K, 1, 1, 1, 0, dt, True, relu)
        dz = dy * (y > 0) if relu else dy
        f64 = lambda a: a.reshape(a.shape[0], -1).astype(np.float64)
        ref = f64(dz) @ f64(w) * (f64(x) > 0)
        with force(tile):
            print("case", dt, (N, C, K), "relu", relu, m.owt_conv_plan_describe(case.desc, 1))
            sys.stdout.flush()
            dx = empty(case.shape_x, dt)
            m.owt_conv_bwd_data_relu_in(case.desc, to_dev(dy, dt), to_dev(y, dt) if relu else None, to_dev(w, dt), to_dev(x, dt), dx, case.ws(1))
            torch.cuda.synchronize()
        got = to_host(dx).reshape(N, C)
        bound = (K / 16 + 16) * 2.0 ** -24 * (np.abs(f64(dz)) @ np.abs(f64(w))) + (2.0 ** -8 * np.abs(ref) if dt == "bf16" else 0.0) + 1e-30
        assert np.max(np.abs(got - ref) / bound) <= 1.0
        assert not got[f64(x) <= 0].any()


def test_split_products_keep_infinities_nans_and_the_ends_of_the_range():
    # an infinite, a NaN and two finite values beyond the largest bf16 among the inputs, tiny values elsewhere: every
    # output is what fp32 products give -- the infinity of the right sign, NaN where a NaN enters, finite otherwise
    m = owt()
    N, C, H, W, K, R, S, pad = shape = (1, 24, 9, 9, 40, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 940)
    x[0, 1, 1, 3], x[0, 1, 6, 9], x[0, 6, 1, 20], x[0, 6, 6, 0] = np.inf, -np.inf, np.nan, np.float32(3.4e38)
    x[0, 4, 4, :] *= np.float32(1e-30)
    x[0, 8, 8, 5] = np.float32(-3.4028234e38)
    w[:, :, :, 0] *= np.float32(0.01)
    with np.errstate(all="ignore"):
        want = np.zeros((H, W, K))
        xp = np.zeros((H + 2, W + 2, C)); xp[1:-1, 1:-1] = x[0]
        for r in range(R):
            for s in range(S):
                want += xp[r:r + H, s:s + W] @ w[:, r, s].astype(np.float64).T
        want = want.astype(np.float32)
    for variant in (0, 2, 3):
        with force(40 + variant, 1):
            got = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", False, False).fwd(x, w, None)[0]
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
        fine = np.isfinite(want)
        assert fine.any() and np.max(np.abs(got[fine] - want[fine]) / (np.abs(want[fine]) + 1e-4 * np.median(np.abs(want[fine])))) < 1e-3


def test_calls_with_the_scratch_of_the_fp32_kernels_still_run():
    # the split filters need workspace; a call that brings none, or too little, is served as it always was
    m = owt()
    N, C, H, W, K, R, S, pad = shape = (2, 32, 13, 13, 64, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 950)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, True)
    assert m.owt_conv_plan_describe(case.desc, 0).startswith("xconv")
    ref = oracle.conv_fwd(x, w, b, 1, pad, True)
    size = oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), 1, pad, False)
    need = m.owt_conv_workspace_bytes(case.desc, 0)
    outs = {}
    for nbytes in (need, 4096, need):
        out = empty(case.shape_y)
        m.owt_conv_fwd(case.desc, to_dev(x), to_dev(w), to_dev(b), out, workspace(nbytes))
        torch.cuda.synchronize()
        outs.setdefault(nbytes, []).append(to_host(out))
        assert np.max(np.abs(outs[nbytes][-1] - ref)) <= 1e-4 * np.max(np.abs(ref))
    check(outs[need][0], ref, size, R * S * C, "y")
    assert np.array_equal(outs[need][0], outs[need][1])
    # with 4 KB it is the kernel that runs where the split ones are switched off, to the bit
    with force(-1, 0, m.OWT_FORCE_NO_BF16_MFMA):
        plan = m.owt_conv_plan_describe(case.desc, 0)
        assert plan.startswith("dconv") and "splitk1 " in plan, plan
        old = case.fwd(x, w, b)
    assert np.array_equal(outs[4096][0], old) and not np.array_equal(old, outs[need][0])


def test_tuning_without_scratch_and_calls_with_unaligned_scratch_still_run():
    # the fp32 kernels need no workspace for this layer: tuning without one, and a pointer the split kernels cannot use
    m = owt()
    N, C, H, W, K, R, S, pad = shape = (1, 8, 6, 7, 8, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 955)
    case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, True)
    ref = oracle.conv_fwd(x, w, b, 1, pad, True)
    out, args = empty(case.shape_y), (to_dev(x), to_dev(w), to_dev(b))
    m.owt_conv_fwd(case.desc, *args, out, workspace(m.owt_conv_workspace_bytes(case.desc, 0) + 16)[4:])
    torch.cuda.synchronize()
    assert np.max(np.abs(to_host(out) - ref)) <= 1e-4 * np.max(np.abs(ref))
    m.owt_conv_autotune(case.desc, 0, *args, out, None, None, None, None)
    assert not m.owt_conv_plan_describe(case.desc, 0).startswith("xconv")
    out.fill_(float("nan"))
    m.owt_conv_fwd(case.desc, *args, out)
    torch.cuda.synchronize()
    assert np.max(np.abs(to_host(out) - ref)) <= 1e-4 * np.max(np.abs(ref))


# N, C, H, W, K, R, S, pad: fewer than 16 images, one more than 16, three groups; ragged filters and channels; rows of one
# and of two positions, filter rows that meet no output row (H = 1), filter height 1, an even number of taps left out by
# the borders, no padding
FILTER_SHAPES = {0: [(16, 40, 13, 13, 136, 3, 3, 1), (1, 5, 1, 1, 3, 3, 3, 1), (17, 33, 7, 2, 70, 3, 3, 1), (5, 8, 9, 6, 12, 1, 3, (0, 1)),
                     (33, 16, 6, 5, 64, 5, 3, (2, 0))],
                 1: [(18, 64, 27, 27, 72, 5, 5, 2), (1, 3, 2, 9, 4, 5, 5, 2), (3, 40, 11, 8, 33, 3, 5, (1, 2)), (16, 32, 6, 5, 32, 5, 5, 0)]}


@pytest.mark.parametrize("variant,split", [(0, 1), (0, 2), (0, 7), (1, 1), (1, 3), (1, 16)])
def test_split_filter_gradient_kernel(variant, split):
    m = owt()
    for i, shape in enumerate(FILTER_SHAPES[variant]):
        N, C, H, W, K, R, S, pad = shape
        x, w, b, dy, y = tensors(shape, 960 + i)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", True, relu)
            g = np.random.default_rng(970 + i)
            dw0 = g.standard_normal(case.shape_w, dtype=np.float32) if beta else None
            db0 = g.standard_normal((K,), dtype=np.float32) if beta else None
            with force(50 + variant, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                print("case", shape, "relu", relu, plan)
                sys.stdout.flush()
                assert plan.startswith("xfilter"), plan
                dw, db = case.bwd_filter(x, dy, y if relu else None, alpha, beta, dw0, db0)
                alone, none = case.bwd_filter(x, dy, y if relu else None, alpha, beta, dw0, db0, want_db=False)
            assert none is None and np.array_equal(alone, dw)
            mask = y if relu else None
            ref, rdb = oracle.conv_bwd_filter(x, dy, (R, S), 1, pad, y=mask, alpha=alpha, beta=beta, dw=dw0, db=db0)
            size, sdb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), 1, pad, y=mask, alpha=alpha, beta=abs(beta),
                                               dw=None if dw0 is None else np.abs(dw0), db=None if db0 is None else np.abs(db0))
            L = N * case.P * case.Q
            check(dw, ref, size, L, "dw")
            check(db, rdb, sdb, L, "db", norm_too=False)


def test_split_filter_gradient_keeps_infinities_nans_and_the_ends_of_the_range():
    # as for the forward pass: the wavefronts whose sums are not finite start over with the careful split
    m = owt()
    N, C, H, W, K, R, S, pad = shape = (3, 40, 6, 7, 70, 3, 3, 1)
    x, w, b, dy, y = tensors(shape, 980)
    x[0, 1, 1, 3], x[1, 5, 6, 9], x[2, 3, 3, 20], x[0, 4, 2, 33] = np.inf, -np.inf, np.nan, np.float32(3.4e38)
    dy[:, :, :, 5] = 0.0                 # inf * 0 is NaN in fp32, too
    dy[1, 2, 2, 7], dy[0, 0, 0, 64] = np.inf, np.float32(-3.4028234e38)
    dy[0, 3:6, 1:4, :] *= np.float32(1e-3)
    with np.errstate(all="ignore"):
        want = np.zeros((K, R, S, C))
        xp = np.zeros((N, H + 2, W + 2, C)); xp[:, 1:-1, 1:-1] = x
        for r in range(R):
            for s in range(S):
                lo = max(0, 1 - r), min(H, H + 1 - r)         # rows of taps outside the image count as zeros, whatever dz holds
                z = dy[:, lo[0]:lo[1]].astype(np.float64)
                cols = max(0, 1 - s), min(W, W + 1 - s)
                want[:, r, s] = np.einsum("nhwk,nhwc->kc", z[:, :, cols[0]:cols[1]],
                                          xp[:, lo[0] + r:lo[1] + r, cols[0] + s:cols[1] + s])
        want = want.astype(np.float32)
    for split in (1, 4):
        with force(50, split):
            got, _ = ConvCase(N, C, H, W, K, R, S, 1, pad, "f32", False, False).bwd_filter(x, dy, None, want_db=False)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
        fine = np.isfinite(want)
        scale = np.median(np.abs(want[fine]))
        assert fine.any() and np.max(np.abs(got[fine].astype(np.float64) - want[fine]) / (np.abs(want[fine]) + 1e-4 * scale)) < 1e-3
        assert np.isinf(got[7]).any() and not np.isfinite(got[7]).any()      # the filter with the infinite dz, at a place that every tap meets


# N, C, H, W, K, R, S, stride, pad: the first layer's geometry on small images (tiles of several images, one per image),
# blocks that hang over every border, strides that differ, a short last chunk, blocks with values past the filter
STRIDED = [(3, 3, 36, 28, 64, 11, 11, 4, 2), (2, 4, 23, 20, 8, 7, 7, 4, 2), (4, 12, 15, 15, 36, 3, 3, 2, 1), (2, 5, 9, 8, 16, 3, 2, (2, 1), (1, 0)),
           (1, 3, 96, 92, 40, 11, 11, 4, 2)]


def strided_tensors(shape, seed):
    N, C, H, W, K, R, S, stride, pad = shape
    g = np.random.default_rng(seed)
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, False)
    return (g.standard_normal(case.shape_x, dtype=np.float32), g.standard_normal(case.shape_w, dtype=np.float32) * np.float32(0.05),
            g.standard_normal((K,), dtype=np.float32), g.standard_normal(case.shape_y, dtype=np.float32),
            g.standard_normal(case.shape_y, dtype=np.float32))


@pytest.mark.parametrize("variant,split", [(1, 1), (3, 1), (1, 2), (3, 3), (0, 1)])
def test_split_strided_forward_over_blocks(variant, split):
    m = owt()
    for i, shape in enumerate(STRIDED):
        N, C, H, W, K, R, S, stride, pad = shape
        x, w, b, dy, y = strided_tensors(shape, 1000 + i)
        case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, True)
        with force(40 + variant, split, m.OWT_FORCE_ONLY_DIRECT):
            plan = m.owt_conv_plan_describe(case.desc, 0)
            print("case", shape, plan)
            sys.stdout.flush()
            assert plan.startswith("sconvx"), plan
            got = case.fwd(x, w, b)
        check(got, oracle.conv_fwd(x, w, b, stride, pad, True), oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), stride, pad, False),
              R * S * C, "y")


def test_split_strided_forward_meets_no_value_outside_its_windows():
    # an infinity and a NaN next to windows, inside the blocks that zero filter values meet: outputs whose windows do not
    # hold them stay finite and exact
    m = owt()
    shape = N, C, H, W, K, R, S, stride, pad = (2, 3, 39, 43, 24, 5, 7, 4, 2)
    x, w, b, dy, y = strided_tensors(shape, 1010)
    ref = oracle.conv_fwd(x, w, b, stride, pad, False)
    bad = np.zeros((N, H, W), bool)
    for n, h, ww, v in ((0, 7, 13, np.inf), (1, 20, 0, np.nan), (1, 38, 42, -np.inf)):
        x[n, h, ww, 1] = v
        bad[n, h, ww] = True
    P, Q = ref.shape[1:3]
    hit = np.zeros((N, P, Q), bool)
    for p in range(P):
        for q in range(Q):
            h0, w0 = p * stride - pad, q * stride - pad
            hit[:, p, q] = bad[:, max(0, h0):h0 + R, max(0, w0):w0 + S].any(axis=(1, 2))
    assert hit.any() and not hit.all()
    for variant, split in ((1, 1), (3, 2)):
        with force(40 + variant, split):
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, False)
            assert owt().owt_conv_plan_describe(case.desc, 0).startswith("sconvx")
            got = case.fwd(x, w, b)
        assert not np.isfinite(got[hit]).any()
        assert np.isfinite(got[~hit]).all() and np.max(np.abs(got[~hit] - ref[~hit])) <= 1e-5 * np.max(np.abs(ref))


def test_split_strided_forward_is_not_held_up_by_values_that_are_not_finite():
    # outputs that are not finite are worked out again one multiply-add at a time: a batch full of NaN or of infinities may take
    # some times as long as a clean one (6 to 9; 39 for one infinity where a wavefront worked its whole tile out again)
    m = owt()
    N, C, H, W, K, R, S, stride, pad = 32, 3, 224, 224, 64, 11, 11, 4, 2
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, True)
    assert m.owt_conv_plan_describe(case.desc, 0).startswith("sconvx")
    g = torch.Generator(device="cuda").manual_seed(1015)
    w, b, y, ws = torch.randn(case.shape_w, generator=g, device="cuda"), torch.randn((K,), generator=g, device="cuda"), empty(case.shape_y), case.ws(0)
    clean = torch.randn(case.shape_x, generator=g, device="cuda")
    one, nans, infs, image = clean.clone(), torch.full_like(clean, float("nan")), torch.full_like(clean, float("inf")), clean.clone()
    one[3, 100, 100, 1] = float("inf")
    image[5] = float("nan")

    def ms(x):
        best = float("inf")
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(3):
                m.owt_conv_fwd(case.desc, x, w, b, y, ws)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) / 3)
        return best

    base = ms(clean)
    for name, x in (("one infinity", one), ("an image of NaN", image), ("all NaN", nans), ("all infinite", infs)):
        t = ms(x)
        print("  clean %.3f ms, %s %.3f ms" % (base, name, t))
        sys.stdout.flush()
        assert t < 16 * base, name


@pytest.mark.parametrize("variant,split", [(0, 1), (0, 3), (1, 1), (1, 7)])
def test_split_filter_gradient_of_any_geometry(variant, split):
    m = owt()
    for i, shape in enumerate(STRIDED + [(17, 5, 6, 7, 70, 3, 3, 1, 1), (8, 3, 12, 12, 16, 5, 5, 1, 2), (1, 1, 8, 8, 1, 3, 3, 1, 1),
                                         (5, 36, 4, 4, 40, 1, 1, 1, 0), (2, 8, 7, 9, 4, 7, 9, 1, 0), (3, 4, 5, 5, 4, 3, 3, 1, 2)]):
        N, C, H, W, K, R, S, stride, pad = shape
        x, w, b, dy, y = strided_tensors(shape, 1020 + i)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, relu)
            g = np.random.default_rng(1040 + i)
            dw0 = g.standard_normal(case.shape_w, dtype=np.float32) if beta else None
            db0 = g.standard_normal((K,), dtype=np.float32) if beta else None
            with force(60 + variant, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                assert plan.startswith(("sfilterx", "xgather")), plan
                print("case", shape, "relu", relu, plan)
                sys.stdout.flush()
                dw, db = case.bwd_filter(x, dy, y if relu else None, alpha, beta, dw0, db0)
            mask = y if relu else None
            ref, rdb = oracle.conv_bwd_filter(x, dy, (R, S), stride, pad, y=mask, alpha=alpha, beta=beta, dw=dw0, db=db0)
            size, sdb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), stride, pad, y=mask, alpha=alpha, beta=abs(beta),
                                               dw=None if dw0 is None else np.abs(dw0), db=None if db0 is None else np.abs(db0))
            L = N * case.P * case.Q
            check(dw, ref, size, L, "dw")
            check(db, rdb, sdb, L, "db", norm_too=False)


# N, C, H, W, K, tile: images of which some past the last would come round to an offset inside the tensor (default plan:
# a kernel that does not address 16 at a time), and tensors of nearly 2^31 bytes whose missing images lie past 2^31 (x, then dz)
@pytest.mark.parametrize("N,C,H,W,K,R,tile", [(3, 16, 2100, 2200, 1, 3, -1), (3, 1, 2100, 2200, 16, 3, -1), (3, 1, 4200, 4300, 4, 5, -1),
                                              (17, 32, 992, 992, 4, 3, 50), (17, 4, 992, 992, 32, 3, 50),
                                              (24, 20, 1000, 1100, 3, 3, 61), (24, 3, 1000, 1100, 20, 3, 61)])
def test_split_filter_gradient_of_large_images(N, C, H, W, K, R, tile):
    m = owt()
    g = torch.Generator(device="cuda").manual_seed(1060)
    x = torch.randn((N, H, W, C), generator=g, device="cuda")
    dy = torch.randn((N, H, W, K), generator=g, device="cuda")
    d = m.conv_desc(N, C, H, W, K, R, R, 1, R // 2, m.OWT_F32, m.OWT_BIAS)
    dw, db = empty((K, R, R, C)), empty((K,))
    with force(tile):
        plan = m.owt_conv_plan_describe(d, 2)
        print("case", (N, C, H, W, K, R), plan)
        sys.stdout.flush()
        assert plan.startswith(("xfilter", "xgather")) == (tile >= 0), plan
        m.owt_conv_bwd_filter(d, x, dy, None, 1.0, 0.0, dw, db, workspace(m.owt_conv_workspace_bytes(d, 2)))
        torch.cuda.synchronize()
    ref, rdb = torch.zeros((K, R, R, C), device="cuda", dtype=torch.float64), torch.zeros((K,), device="cuda", dtype=torch.float64)
    pad = R // 2
    for n in range(N):
        xp = torch.zeros((H + 2 * pad, W + 2 * pad, C), device="cuda", dtype=torch.float64)
        xp[pad:pad + H, pad:pad + W] = x[n]
        z = dy[n].double().view(-1, K)
        rdb += z.sum(0)
        for r in range(R):
            for s in range(R):
                xs = xp[r:r + H, s:s + W].reshape(-1, C)
                if K < C:                                         # (a product this long and narrow is slow)
                    ref[:, r, s] += torch.stack([(xs * z[:, k:k + 1]).sum(0) for k in range(K)])
                else:
                    ref[:, r, s] += torch.stack([(z * xs[:, c:c + 1]).sum(0) for c in range(C)], 1)
    # sums of L products of independent normal values are sqrt(L) large and their rounding errors at most 2^-24 sqrt(L) each
    # time a partial sum is rounded, L/16 times at random: 2^-24 L/4 absolute.  One image too many moves them by sqrt(L/N).
    L = N * H * W
    bound = max(2.0 ** -24 * L / 4, 1e-3)
    assert bound < 0.1 * np.sqrt(L / N)
    assert (dw - ref).abs().max().item() <= bound and (db - rdb).abs().max().item() <= bound
    print("  largest error %.3f and %.3f of the bound" % ((dw - ref).abs().max().item() / bound, (db - rdb).abs().max().item() / bound))


# N, I, O: single values, one step and tile less, exactly and more than full, odd rows (2-byte aligned in bf16), more tiles
# than CUs
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("split", [1, 3])
def test_fully_connected_shard_on_the_bf16_matrix_unit(dt, split):
    m = owt()
    rnd = oracle.round_bf16 if dt == "bf16" else (lambda a: a)
    code = m.OWT_BF16 if dt == "bf16" else m.OWT_F32
    for i, (N, I, O) in enumerate([(1, 1, 1), (5, 17, 3), (16, 64, 64), (33, 100, 65), (64, 16, 128), (130, 131, 70), (20, 5000, 260)]):
        g = np.random.default_rng(1100 + i)
        x, w = rnd(g.standard_normal((N, I), dtype=np.float32)), rnd(g.standard_normal((O, I), dtype=np.float32) * np.float32(0.05))
        b, dy, y = g.standard_normal((O,), dtype=np.float32), rnd(g.standard_normal((N, O), dtype=np.float32)), rnd(g.standard_normal((N, O), dtype=np.float32))
        dw0, db0 = g.standard_normal((O, I), dtype=np.float32), g.standard_normal((O,), dtype=np.float32)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            d = m.fc_desc(N, I, O, 1, 0, code, m.OWT_BIAS | (m.OWT_RELU if relu else 0))
            yin = y if relu else None
            with force(70, split):
                print("case", dt, (N, I, O), "relu", relu, "split", split)
                sys.stdout.flush()
                ws = workspace(max(m.owt_fc_workspace_bytes(d, 0), m.owt_fc_workspace_bytes(d, 1)))
                yd, dx, dw, db = empty((N, O), dt), empty((N, I), dt), to_dev(dw0), to_dev(db0)
                m.owt_fc_shard_fwd(d, to_dev(x, dt), to_dev(w, dt), to_dev(b), yd, ws)
                m.owt_fc_shard_bwd(d, to_dev(x, dt), to_dev(w, dt), to_dev(yin, dt), to_dev(dy, dt), alpha, beta, dx, dw, db, ws)
                dw2 = to_dev(dw0)
                m.owt_fc_shard_bwd(d, to_dev(x, dt), to_dev(w, dt), to_dev(yin, dt), to_dev(dy, dt), alpha, beta, None, dw2, None, ws)
                torch.cuda.synchronize()
            assert torch.equal(dw, dw2)
            dz = dy * (y > 0) if relu else dy
            f64 = lambda a: a.astype(np.float64)
            lin = f64(x) @ f64(w).T + b
            refs = {"y": (to_host(yd), np.maximum(lin, 0) if relu else lin, np.abs(f64(x)) @ np.abs(f64(w)).T + np.abs(b), I),
                    "dx": (to_host(dx), f64(dz) @ f64(w), np.abs(f64(dz)) @ np.abs(f64(w)), O),
                    "dw": (to_host(dw), alpha * (f64(dz).T @ f64(x)) + beta * dw0, abs(alpha) * (np.abs(f64(dz)).T @ np.abs(f64(x))) + abs(beta) * np.abs(dw0), N),
                    "db": (to_host(db), alpha * f64(dz).sum(0) + beta * db0, abs(alpha) * np.abs(f64(dz)).sum(0) + abs(beta) * np.abs(db0), N)}
            for name, (got, ref, size, L) in refs.items():
                bound = (L / 16 + 16) * 2.0 ** -24 * size + 1e-30
                if dt == "bf16" and name in ("y", "dx"):
                    bound += 2.0 ** -8 * np.abs(ref)              # rounded to bf16 when stored
                worst = np.max(np.abs(got - ref) / bound)
                assert worst <= 1.0, (name, worst)


# tuned: whichever way of running the two backward products was the fastest (one launch on the bf16 matrix unit, the dense
# kernel in one or two, each a pass of its own) gives the results; tuned twice, and the products tuned alone in between
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N,I,O", [(128, 512, 512), (29, 868, 499), (130, 131, 70), (256, 4096, 64), (2, 103, 41)])
def test_tuned_shard_backward(dt, N, I, O):
    m = owt()
    rnd = oracle.round_bf16 if dt == "bf16" else (lambda a: a)
    g = np.random.default_rng(1150)
    x, w = rnd(g.standard_normal((N, I), dtype=np.float32)), rnd(g.standard_normal((O, I), dtype=np.float32) * np.float32(0.05))
    dy, y = rnd(g.standard_normal((N, O), dtype=np.float32)), rnd(g.standard_normal((N, O), dtype=np.float32))
    code = m.OWT_BF16 if dt == "bf16" else m.OWT_F32
    d = m.fc_desc(N, I, O, 1, 0, code, m.OWT_RELU)
    c = m.conv_desc(N, I, 1, 1, O, 1, 1, 1, 0, code, m.OWT_RELU)
    ws = workspace(max(m.owt_fc_workspace_bytes(d, 0), m.owt_fc_workspace_bytes(d, 1)))
    xd, wd, yd, dyd = to_dev(x, dt), to_dev(w, dt), to_dev(y, dt), to_dev(dy, dt)
    f64 = lambda a: a.astype(np.float64)
    dz = f64(dy) * (y > 0)
    refs = {"dx": (dz @ f64(w), np.abs(dz) @ np.abs(f64(w)), O), "dw": (dz.T @ f64(x), np.abs(dz).T @ np.abs(f64(x)), N), "db": (dz.sum(0), np.abs(dz).sum(0), N)}
    for again in range(3):
        out = {"dx": empty((N, I), dt), "dw": empty((O, I)), "db": empty((O,))}
        if again == 2:
            for p in (1, 2):
                m.owt_conv_autotune(c, p, xd, wd, None, yd, dyd, out["dx"], out["dw"], out["db"], ws)
        else:
            m.owt_fc_autotune(d, xd, wd, None, empty((N, O), dt), dyd, out["dx"], out["dw"], out["db"], ws)
        for t in out.values():
            t.fill_(float("nan"))
        m.owt_fc_shard_bwd(d, xd, wd, yd, dyd, 1.0, 0.0, out["dx"], out["dw"], out["db"], ws)
        torch.cuda.synchronize()
        for name, (ref, size, L) in refs.items():
            bound = (L / 2 + 16) * 2.0 ** -24 * size + 1e-30        # the fp32 instruction rounds every second product
            if dt == "bf16" and name == "dx":
                bound += 2.0 ** -8 * np.abs(ref)
            assert np.max(np.abs(to_host(out[name]) - ref) / bound) <= 1.0, (name, again)


# Operands at the ends of the fp32 range: (scale of the one, of the other) with results well inside it.  2^-118: normal and
# subnormal values; 2^106 next to 2^-100; sums near 2^100 of operands near 2^50.  Every bit of an operand counts: the 2-norm bound
# of the ordinary range has to hold (a sum beyond 2^80 may be an fp32 sum in order, whose roundings are L at random).
ENDS = [(2.0 ** -118, 2.0 ** 20), (2.0 ** 20, 2.0 ** -118), (2.0 ** 106, 2.0 ** -100), (2.0 ** -100, 2.0 ** 106), (2.0 ** 50, 2.0 ** 50), (2.0 ** -60, 2.0 ** -50)]


def check_ends(got, ref, L, what):
    norm = np.linalg.norm((got - ref) / np.abs(ref).max()) / np.linalg.norm(ref / np.abs(ref).max())
    bound = 2.0 ** -23 * np.sqrt((L if np.abs(ref).max() > 2.0 ** 79 else L / 16) + 4)
    print("  %s: relative 2-norm error %.2e of %.2e" % (what, norm, bound))
    sys.stdout.flush()
    assert norm <= bound, what


def conv64(x, w, stride, pad, P, Q):
    (N, H, W, C), (K, R, S, _) = x.shape, w.shape
    xp = np.zeros((N, H + 2 * pad, W + 2 * pad, C)); xp[:, pad:pad + H, pad:pad + W] = x
    y, dw_of = np.zeros((N, P, Q, K)), []
    for r in range(R):
        for s in range(S):
            xs = xp[:, r:r + (P - 1) * stride + 1:stride, s:s + (Q - 1) * stride + 1:stride]
            y += xs @ w[:, r, s].astype(np.float64).T
            dw_of.append((r, s, xs))
    return y, dw_of


@pytest.mark.parametrize("a,b", ENDS)
def test_split_kernels_at_the_ends_of_the_range(a, b):
    m = owt()
    with np.errstate(under="ignore"):
        for tiles, shape in (((40, 41, 42, 43), (2, 24, 9, 10, 40, 3, 3, 1, 1)), ((41, 43), (2, 3, 39, 43, 24, 5, 7, 4, 2))):
            N, C, H, W, K, R, S, stride, pad = shape
            g = np.random.default_rng(1200)
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)
            x = (g.standard_normal(case.shape_x) * a).astype(np.float32)
            w = (g.standard_normal(case.shape_w) * b).astype(np.float32)
            ref = conv64(x, w, stride, pad, case.P, case.Q)[0]
            for tile in tiles:
                for split in (1, 2):
                    with force(tile, split):
                        plan = m.owt_conv_plan_describe(case.desc, 0)
                        assert plan.startswith(("xconv", "sconvx")), plan
                        check_ends(case.fwd(x, w, None), ref, R * S * C, "y " + plan)
            if stride == 1:           # dx of a symmetric layer is a forward pass with the filters turned round
                dy = (g.standard_normal(case.shape_y) * a).astype(np.float32)
                y = g.standard_normal(case.shape_y).astype(np.float32)
                masked = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, True)
                ref = conv64(dy * (y > 0), w[:, ::-1, ::-1].transpose(3, 1, 2, 0), 1, pad, H, W)[0]
                for tile in tiles:
                    for split in (1, 2):
                        with force(tile, split):
                            check_ends(masked.bwd_data(dy, y, w), ref, R * S * K, "dx")
        for tile, shape in ((50, (18, 40, 6, 7, 70, 3, 3, 1, 1)), (51, (18, 40, 6, 7, 33, 5, 5, 1, 2)), (60, (18, 3, 23, 20, 64, 7, 7, 4, 2)), (61, (18, 3, 23, 20, 30, 7, 7, 4, 2))):
            N, C, H, W, K, R, S, stride, pad = shape
            g = np.random.default_rng(1210)
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)
            x = (g.standard_normal(case.shape_x) * a).astype(np.float32)
            dy = (g.standard_normal(case.shape_y) * b).astype(np.float32)
            ref = np.zeros(case.shape_w)
            for r, s, xs in conv64(x, np.zeros(case.shape_w), stride, pad, case.P, case.Q)[1]:
                ref[:, r, s] = dy.reshape(-1, K).astype(np.float64).T @ xs.reshape(-1, C)
            for split in (1, 3):
                with force(tile, split):
                    plan = m.owt_conv_plan_describe(case.desc, 2)
                    assert plan.startswith(("xfilter", "xgather", "sfilterx")), plan
                    check_ends(case.bwd_filter(x, dy, None, want_db=False)[0], ref, N * case.P * case.Q, "dw " + plan)
        N, I, O = 70, 300, 90
        g = np.random.default_rng(1220)
        x, w, dy = ((g.standard_normal(sh) * sc).astype(np.float32) for sh, sc in (((N, I), a), ((O, I), b), ((N, O), b)))
        d = m.fc_desc(N, I, O, 1, 0, m.OWT_F32, 0)
        d2 = m.fc_desc(N, O, I, 1, 0, m.OWT_F32, 0)            # its backward pass: dx and dw of operands scaled a and b, too
        f64 = lambda t: t.astype(np.float64)
        for split in (1, 2):
            with force(70, split):
                ws = workspace(max(m.owt_fc_workspace_bytes(q, p) for q in (d, d2) for p in (0, 1)))
                y, dx, dw = empty((N, O)), empty((N, O)), empty((I, O))
                m.owt_fc_shard_fwd(d, to_dev(x), to_dev(w), None, y, ws)
                # layer O -> I: its dy is x (N, I), its weights w.T (I, O), its input dy (N, O)
                m.owt_fc_shard_bwd(d2, to_dev(dy), to_dev(np.ascontiguousarray(w.T)), None, to_dev(x), 1.0, 0.0, dx, dw, None, ws)
                torch.cuda.synchronize()
            check_ends(to_host(y), f64(x) @ f64(w).T, I, "shard y")
            check_ends(to_host(dx), f64(x) @ f64(w).T, I, "shard dx")
            check_ends(to_host(dw), f64(x).T @ f64(dy), N, "shard dw")


def test_a_product_just_below_the_largest_number_stays_finite():
    # 0x1.ffp0 * 0x1.ffp126 = 0x1.fe01p127, each operand halfway between two bf16 values: their large parts alone give 2^128
    m = owt()
    one, big = np.float32(float.fromhex("0x1.ffp0")), np.float32(float.fromhex("0x1.ffp126"))
    want = np.float32(float(one) * float(big))
    assert np.isfinite(want)
    for u, v in ((one, big), (big, one), (-one, big)):
        want = np.float32(float(u) * float(v))
        for tile, shape in ((40, (1, 20, 5, 6, 9, 3, 3, 1, 1)), (42, (1, 20, 5, 6, 9, 1, 1, 1, 0)), (43, (1, 20, 5, 6, 9, 3, 3, 1, 1)), (41, (1, 3, 24, 24, 9, 5, 5, 4, 2))):
            N, C, H, W, K, R, S, stride, pad = shape
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)
            x, w = np.zeros(case.shape_x, np.float32), np.zeros(case.shape_w, np.float32)
            x[0, 2, 2, 2] = u
            w[4, R // 2, S // 2, 2] = v
            with force(tile, 1):
                got = case.fwd(x, w, None)
            ref = conv64(x, w, stride, pad, case.P, case.Q)[0].astype(np.float32)
            assert np.abs(ref).max() == abs(want) or stride > 1
            assert np.array_equal(got, ref), (tile, got[np.abs(got) > 0], want)
        for tile, shape in ((50, (3, 5, 4, 5, 9, 3, 3, 1, 1)), (51, (3, 5, 4, 5, 9, 5, 5, 1, 2)), (61, (3, 3, 9, 9, 9, 3, 3, 2, 1))):
            N, C, H, W, K, R, S, stride, pad = shape
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)
            x, dy = np.zeros(case.shape_x, np.float32), np.zeros(case.shape_y, np.float32)
            x[1, 2, 2, 1], dy[1, 1, 1, 3] = u, v
            ref = np.zeros(case.shape_w)
            for r, s, xs in conv64(x, np.zeros(case.shape_w), stride, pad, case.P, case.Q)[1]:
                ref[:, r, s] = dy.reshape(-1, K).astype(np.float64).T @ xs.reshape(-1, C)
            assert np.abs(ref).max() == abs(float(u) * float(v))
            with force(tile, 1):
                got, _ = case.bwd_filter(x, dy, None, want_db=False)
            assert np.array_equal(got, ref.astype(np.float32)), tile
        for split in (1, 2):
            N, I, O = 5, 40, 7
            x, w = np.zeros((N, I), np.float32), np.zeros((O, I), np.float32)
            x[2, 3], w[4, 3] = u, v
            d = m.fc_desc(N, I, O, 1, 0, m.OWT_F32, 0)
            with force(70, split):
                ws, y = workspace(m.owt_fc_workspace_bytes(d, 0)), empty((N, O))
                m.owt_fc_shard_fwd(d, to_dev(x), to_dev(w), None, y, ws)
                torch.cuda.synchronize()
            assert np.array_equal(to_host(y), (x.astype(np.float64) @ w.astype(np.float64).T).astype(np.float32))


@pytest.mark.parametrize("tile,shape", [(50, (128, 32, 13, 13, 384, 3, 3, 1, 1)), (50, (2, 32, 39, 46, 64, 3, 3, 1, 1)), (60, (64, 3, 55, 55, 64, 3, 3, 2, 1)), (61, (128, 4, 13, 13, 384, 3, 3, 1, 1))])
def test_split_bias_gradient_is_no_single_chain(tile, shape):
    # Sums of n normal values are sqrt(n) large, and an addition rounds by 0.29 * 2^-23 of its result (2-norm), at random.  Eight
    # images in a tree: 7/8 n results of 3 squared; rows of L positions (or runs of L = 16): n/8 results of up to 8 L / 2; the whole:
    # n / (8 L) results of n / 2.  Half as much again is allowed.  One chain of all positions has n/8 results of n / 2.
    m = owt()
    N, C, H, W, K, R, S, stride, pad = shape
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, False)
    g = torch.Generator(device="cuda").manual_seed(1250)
    worst = 0.0
    for seed in range(4):
        x, dy = torch.randn(case.shape_x, generator=g, device="cuda"), torch.randn(case.shape_y, generator=g, device="cuda")
        dw, db = empty(case.shape_w), empty((K,))
        with force(tile, 1):
            assert m.owt_conv_plan_describe(case.desc, 2).startswith(("xfilter", "xgather", "sfilterx"))
            m.owt_conv_bwd_filter(case.desc, x, dy, None, 1.0, 0.0, dw, db, case.ws(2))
            torch.cuda.synchronize()
        ref = dy.double().view(-1, K).sum(0)
        worst = max(worst, ((db - ref).norm() / ref.norm()).item())
    n, L = N * case.P * case.Q, case.Q if tile < 60 else 16
    bound = 1.5 * 0.29 * np.sqrt(7 / 8 * 3 + L / 2 + n / (16 * L))
    print("  worst of four: %.2f * 2^-23 of %.2f" % (worst * 2 ** 23, bound))
    assert worst * 2 ** 23 < bound < 1.5 * 0.29 * np.sqrt(n / 16)


# tensors of nearly 2^31 bytes: x, then y, of a forward pass (dy and dx of a backward-data pass are the same kernel's), x of a strided
# one, and both operands of the shard; the first and last images or rows against 64 bits
@pytest.mark.parametrize("N,C,H,W,K,R,stride,pad,tile", [(2000, 64, 64, 65, 9, 3, 1, 1, 41), (2000, 9, 64, 65, 64, 3, 1, 1, 43), (3500, 3, 224, 224, 8, 11, 4, 2, 43)])
def test_split_convolution_of_large_tensors(N, C, H, W, K, R, stride, pad, tile):
    m = owt()
    g = torch.Generator(device="cuda").manual_seed(1300)
    case = ConvCase(N, C, H, W, K, R, R, stride, pad, "f32", False, False)
    assert 2 ** 31 - 2 ** 26 < 4 * max(np.prod(case.shape_x), np.prod(case.shape_y)) < 2 ** 31
    x, w = torch.randn(case.shape_x, generator=g, device="cuda"), torch.randn(case.shape_w, generator=g, device="cuda")

    def ref(a, wt, st, pd, P, Q):
        ap = torch.zeros((a.shape[0], a.shape[1] + 2 * pd, a.shape[2] + 2 * pd, a.shape[3]), device="cuda", dtype=torch.float64)
        ap[:, pd:pd + a.shape[1], pd:pd + a.shape[2]] = a
        out = 0
        for r in range(R):
            for s in range(R):
                out = out + ap[:, r:r + (P - 1) * st + 1:st, s:s + (Q - 1) * st + 1:st].reshape(-1, a.shape[3]) @ wt[:, r, s].double().t().contiguous()
        return out.view(a.shape[0], P, Q, -1)

    ends = [0, 1, N - 2, N - 1]
    bound = (R * R * C / 16 + 16) * 2.0 ** -24 * R * R * C
    with force(tile):
        print("case", case.shape_x, case.shape_y, m.owt_conv_plan_describe(case.desc, 0))
        sys.stdout.flush()
        assert m.owt_conv_plan_describe(case.desc, 0).startswith(("xconv", "sconvx"))
        y = empty(case.shape_y)
        m.owt_conv_fwd(case.desc, x, w, None, y, case.ws(0))
        torch.cuda.synchronize()
    assert (y[ends] - ref(x[ends], w, stride, pad, case.P, case.Q)).abs().max().item() < bound
    if stride == 1:
        dx = empty(case.shape_x)
        with force(tile):
            assert m.owt_conv_plan_describe(case.desc, 1).startswith("xconv")
            m.owt_conv_bwd_data_relu_in(case.desc, y, None, w, x, dx, case.ws(1))
            torch.cuda.synchronize()
        want = ref(y[ends], w.flip(1, 2).permute(3, 1, 2, 0).contiguous(), 1, pad, H, W) * (x[ends] > 0)
        size = (R * R * C) ** 0.5                                # of the values in y
        assert (dx[ends] - want).abs().max().item() < (R * R * K / 16 + 16) * 2.0 ** -24 * R * R * K * size


@pytest.mark.parametrize("N,I,O", [(60000, 8900, 24), (40, 8900, 60000)])
def test_fully_connected_shard_of_large_tensors(N, I, O):
    m = owt()
    g = torch.Generator(device="cuda").manual_seed(1310)
    x, w, dy = (torch.randn(s, generator=g, device="cuda") for s in ((N, I), (O, I), (N, O)))
    d = m.fc_desc(N, I, O, 1, 0, m.OWT_F32, 0)
    with force(70):
        ws = workspace(max(m.owt_fc_workspace_bytes(d, 0), m.owt_fc_workspace_bytes(d, 1)))
        y, dx, dw = empty((N, O)), empty((N, I)), empty((O, I))
        m.owt_fc_shard_fwd(d, x, w, None, y, ws)
        m.owt_fc_shard_bwd(d, x, w, None, dy, 1.0, 0.0, dx, dw, None, ws)
        torch.cuda.synchronize()
    n, o = [0, 1, N - 2, N - 1], [0, 1, O - 2, O - 1]
    f64 = lambda t: t.double()
    for name, got, want, L in (("y", y[n], f64(x[n]) @ f64(w).t(), I), ("dx", dx[n], f64(dy[n]) @ f64(w), O), ("dw", dw[o], f64(dy[:, o]).t() @ f64(x), N)):
        err = ((got - want).norm() / want.norm()).item()
        print("  %s: %.2e" % (name, err))
        assert err < 2.0 ** -23 * np.sqrt(L / 16 + 4), name


@pytest.mark.parametrize("tile,shape", [(50, (18, 40, 6, 7, 70, 3, 3, 1, 1)), (51, (18, 40, 6, 7, 33, 5, 5, 1, 2)), (60, (18, 3, 23, 20, 64, 7, 7, 4, 2)), (61, (18, 3, 23, 20, 30, 7, 7, 4, 2))])
def test_both_ends_of_the_range_in_one_tile(tile, shape):
    # channel 0 near 2^110, where scaled operands are infinite, channel 1 near 2^-118: the tile's second run is not finite, its third
    # keeps 2^-13 of channel 1 (a part of 2^-118 that bf16 still holds is 2^-133, 2^-15 of it), everything of the others
    m = owt()
    N, C, H, W, K, R, S, stride, pad = shape
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)
    g = np.random.default_rng(1230)
    x, dy = g.standard_normal(case.shape_x), g.standard_normal(case.shape_y)
    x[..., 0] *= 2.0 ** 110
    x[..., 1] *= 2.0 ** -118
    x, dy = x.astype(np.float32), dy.astype(np.float32)
    ref = np.zeros(case.shape_w)
    for r, s, xs in conv64(x, np.zeros(case.shape_w), stride, pad, case.P, case.Q)[1]:
        ref[:, r, s] = dy.reshape(-1, K).astype(np.float64).T @ xs.reshape(-1, C)
    for split in (1, 3):
        with force(tile, split):
            assert m.owt_conv_plan_describe(case.desc, 2).startswith(("xfilter", "xgather", "sfilterx"))
            got = case.bwd_filter(x, dy, None, want_db=False)[0]
        assert np.isfinite(got).all()
        check_ends(got[..., 0], ref[..., 0], N * case.P * case.Q, "channel 0")
        check_ends(got[..., 2:], ref[..., 2:], N * case.P * case.Q, "the others")
        low = np.linalg.norm((got[..., 1] - ref[..., 1]) * 2.0 ** 118) / np.linalg.norm(ref[..., 1] * 2.0 ** 118)
        print("  channel 1: %.2e" % low)
        assert low < 2.0 ** -13
