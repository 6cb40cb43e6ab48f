"""The planner's choices and refusals, without a GPU: which kernel a geometry gets, what a call with little scratch is
served by, what the workspace queries ask for."""
import ctypes
import time

import pytest


@pytest.fixture(scope="module")
def m():
    import paper_1404_5997_amd as mod
    return mod


def plan(m, shape, p, relu=False, dtype=0):
    N, C, H, W, K, R, S, stride, pad = shape
    return m.owt_conv_plan_describe(m.conv_desc(N, C, H, W, K, R, S, stride, pad, dtype, m.OWT_BIAS | (m.OWT_RELU if relu else 0)), p)


def wraps(images, image_bytes, all_bytes):
    """Does an image past the last, addressed in 32 bits, land inside the tensor again?"""
    return any((n * image_bytes) % 2 ** 32 < all_bytes for n in range(images, 16 * ((images + 15) // 16)))


# N, C, H, W, K, R, S, stride, pad: images of more than 2^32 / 15 bytes, where some image of the last group of 16 comes round
WRAPPING = [(7, 64, 1024, 1100, 64, 3, 3, 1, 1), (6, 64, 1152, 1152, 64, 3, 3, 1, 1), (5, 64, 1280, 1280, 64, 3, 3, 1, 1),
            (4, 64, 1408, 1408, 64, 3, 3, 1, 1), (7, 128, 768, 768, 128, 3, 3, 1, 1), (7, 512, 384, 384, 512, 3, 3, 1, 1),
            (3, 37, 2100, 2100, 37, 3, 3, 1, 1), (7, 64, 1080, 1080, 64, 1, 1, 1, 0), (4, 32, 1536, 1500, 32, 3, 3, 1, 1),
            (3, 10, 4000, 4000, 10, 3, 3, 1, 1), (7, 2, 1080, 1080, 64, 3, 3, 1, 1), (7, 64, 1080, 1080, 2, 3, 3, 1, 1),
            (2, 3, 6000, 6000, 7, 5, 5, 1, 2)]


@pytest.mark.parametrize("shape", WRAPPING)
def test_large_images_stay_off_the_kernels_that_address_16_at_a_time(m, shape):
    N, C, H, W, K, R, S, stride, pad = shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    assert wraps(N, H * W * C * 4, N * H * W * C * 4) or wraps(N, P * Q * K * 4, N * P * Q * K * 4)
    for relu in (False, True):
        for tile in (-1, 50, 51, 60, 61):
            m.owt_test_force_variant(tile, 0, 0)
            try:
                p = plan(m, shape, 2, relu)
            finally:
                m.owt_test_force_variant(-1, 0, 0)
            assert not p.startswith(("xfilter", "xgather", "sfilterx")), (tile, p)


def test_images_that_do_not_wrap_keep_those_kernels(m):
    for tile, kernel, shape in ((50, "xfilter", (8, 64, 1000, 1040, 64, 3, 3, 1, 1)), (50, "xfilter", (1, 64, 1000, 1040, 64, 3, 3, 1, 1)),
                                (50, "xfilter", (17, 32, 992, 992, 4, 3, 3, 1, 1)), (60, "xgather", (24, 32, 800, 860, 32, 3, 3, 1, 1)),
                                (61, "xgather", (16, 5, 2000, 2100, 7, 3, 3, 1, 1))):
        N, C, H, W, K = shape[:5]
        assert not wraps(N, H * W * C * 4, N * H * W * C * 4) and not wraps(N, H * W * K * 4, N * H * W * K * 4)
        m.owt_test_force_variant(tile, 0, 0)
        try:
            assert plan(m, shape, 2).startswith(kernel), shape
        finally:
            m.owt_test_force_variant(-1, 0, 0)
    assert plan(m, (8, 64, 1000, 1040, 64, 3, 3, 1, 1), 2).startswith("xfilter")


# the same for the variants whose four wavefronts share a tile
@pytest.mark.parametrize("tile", [52, 53, 62, 63])
def test_large_images_stay_off_the_shared_tiles(m, tile):
    for shape in WRAPPING + [(8, 64, 1000, 1040, 64, 3, 3, 1, 1), (8, 64, 1000, 1040, 64, 5, 5, 1, 2)]:
        m.owt_test_force_variant(tile, 0, 0)
        try:
            p = plan(m, shape, 2)
        finally:
            m.owt_test_force_variant(-1, 0, 0)
        takes = shape not in WRAPPING and (tile > 60 or shape[6] == (3 if tile == 52 else 5))
        if not takes:
            assert not p.startswith(("xfilter", "xgather", "sfilterx")), (shape, p)
        elif tile < 60:                                # (xgather's line is a little lower)
            assert p.startswith("xfilter"), (shape, p)


# bf16 storage: the same images in bytes with twice the channels
@pytest.mark.parametrize("shape", WRAPPING)
def test_large_bf16_images_stay_off_the_kernels_that_address_16_at_a_time(m, shape):
    N, C, H, W, K, R, S, stride, pad = shape
    shape = (N, 2 * C, H, W, 2 * K, R, S, stride, pad)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    assert wraps(N, H * W * C * 4, N * H * W * C * 4) or wraps(N, P * Q * K * 4, N * P * Q * K * 4)
    for relu in (False, True):
        for tile in [-1] + list(range(80, 87)) + [88, 89]:
            m.owt_test_force_variant(tile, 0, 0)
            try:
                p = plan(m, shape, 2, relu, dtype=1)
            finally:
                m.owt_test_force_variant(-1, 0, 0)
            assert not p.startswith(("ifilter16", "igather16", "sfilter16x")), (tile, p)


# just below the line that such an image crosses: tile, kernel, shape
@pytest.mark.parametrize("tile,kernel,shape", [
    (80, "ifilter16", (8, 128, 1000, 1040, 128, 3, 3, 1, 1)), (83, "ifilter16", (1, 128, 1000, 1040, 128, 3, 3, 1, 1)), (82, "ifilter16", (17, 64, 992, 992, 8, 3, 3, 1, 1)),
    (84, "ifilter16", (7, 37, 1100, 1300, 45, 5, 5, 1, 2)), (88, "igather16", (24, 64, 800, 860, 64, 3, 3, 1, 1)), (89, "igather16", (16, 10, 2000, 2100, 14, 3, 3, 1, 1)),
    (89, "sfilter16x", (16, 10, 2000, 2100, 14, 3, 3, 2, 1)), (-1, "ifilter16", (8, 128, 1000, 1040, 128, 3, 3, 1, 1))])
def test_bf16_images_that_do_not_wrap_keep_those_kernels(m, tile, kernel, shape):
    N, C, H, W, K, R, S, stride, pad = shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    assert not wraps(N, H * W * C * 2, N * H * W * C * 2) and not wraps(N, P * Q * K * 2, N * P * Q * K * 2)
    m.owt_test_force_variant(tile, 0, 0)
    try:
        assert plan(m, shape, 2, dtype=1).startswith(kernel), shape
    finally:
        m.owt_test_force_variant(-1, 0, 0)


# the filter gradient over images with streamed operands: the same line, on either side of it, and what it does not take
@pytest.mark.parametrize("tile,S", [(100, 3), (103, 3), (104, 5), (106, 5)])
def test_streamed_images_keep_to_what_they_can_address(m, tile, S):
    def name(shape, relu=False):
        m.owt_test_force_variant(tile, 0, 0)
        try:
            return plan(m, shape, 2, relu, dtype=1)
        finally:
            m.owt_test_force_variant(-1, 0, 0)
    for shape in WRAPPING:
        N, C, H, W, K, R, _, stride, pad = shape
        assert not name((N, (2 * C + 7) // 8 * 8, H, W, (2 * K + 7) // 8 * 8, S, S, 1, S // 2)).startswith("ifilter16b"), shape
    for shape in ((8, 128, 1000, 1040, 128), (1, 128, 1000, 1040, 128), (17, 64, 992, 992, 8)):
        N, C, H, W, K = shape
        assert not wraps(N, H * W * C * 2, N * H * W * C * 2) and not wraps(N, H * W * K * 2, N * H * W * K * 2)
        assert name(shape + (S, S, 1, S // 2)).startswith("ifilter16b"), shape
    takes = (9, 64, 20, 24, 32, S, S, 1, S // 2)
    assert name(takes).startswith("ifilter16b")
    for other in ((9, 60, 20, 24, 32, S, S, 1, S // 2), (9, 64, 20, 24, 36, S, S, 1, S // 2), (9, 64, 20, 24, 32, S, S, 2, S // 2)):
        assert not name(other).startswith("ifilter16b"), other
    assert not name(takes, relu=True).startswith("ifilter16b")


# and it stores dw with 32-bit byte offsets: filters of up to 2 GB, rows of a ragged tile included (256, 128 and 64 filters)
@pytest.mark.parametrize("tile,S,K,C", [(None, 3, 8200, 8200), (None, 3, 12000, 12000), (None, 3, 7680, 7768), (100, 3, 8200, 8200), (100, 3, 7680, 7768),
                                        (103, 3, 7736, 7640), (104, 5, 5184, 4144), (106, 5, 4672, 4608), (106, 5, 4600, 4680), (103, 3, 8, 466040)])
def test_streamed_images_leave_filters_that_they_cannot_address(m, tile, S, K, C):
    shape = (16, C, 6 if C < 100000 else 3, 6 if C < 100000 else 3, K, S, S, 1, S // 2)
    m.owt_test_force_variant(-1 if tile is None else tile, 0, 0)
    try:
        assert not plan(m, shape, 2, dtype=1).startswith("ifilter16b"), shape
    finally:
        m.owt_test_force_variant(-1, 0, 0)


@pytest.mark.parametrize("tile,S,K,C", [(100, 3, 7680, 7760), (103, 3, 7736, 7632), (104, 5, 5184, 4136), (106, 5, 4608, 4656), (103, 3, 8, 466032)])
def test_streamed_images_take_filters_up_to_that_line(m, tile, S, K, C):
    m.owt_test_force_variant(tile, 0, 0)
    try:
        assert plan(m, (16, C, 6 if C < 100000 else 3, 6 if C < 100000 else 3, K, S, S, 1, S // 2), 2, dtype=1).startswith("ifilter16b"), (K, C)
    finally:
        m.owt_test_force_variant(-1, 0, 0)


# the bf16 kernels with 32-bit byte offsets: tensors below 2 GB, and below 1 GB for the one of few tiles, whose partial sums take 4 bytes
@pytest.mark.parametrize("tile,kernel,images,p", [(90, "dconv16x", 8061, 0), (90, "dconv16x", 8061, 1), (92, "dconv16s", 4030, 0), (94, "dconv16s", 4030, 1)])
@pytest.mark.parametrize("C,K", [(37, 5), (5, 37)])
def test_bf16_tensors_past_32_bit_offsets_stay_off_the_kernels_that_use_them(m, tile, kernel, images, p, C, K):
    for n, takes in ((images, True), (images + 1, False)):
        m.owt_test_force_variant(tile, 1, 0)
        try:
            name = plan(m, (n, C, 60, 60, K, 3, 3, 1, 1), p, dtype=1)
        finally:
            m.owt_test_force_variant(-1, 0, 0)
        assert name.startswith(kernel) == takes, (n, name)


# the 1x1 filter has no kernel but those and the gather kernel, which flag 2 (only the direct kernels) leaves out
@pytest.mark.parametrize("tile,flags,shape", [(t, 0, (2, 32, 13, 13, 64, 3, 3, 1, 1)) for t in (40, 41, 43, 50, 61)] +
                         [(40, 2, (2, 32, 13, 13, 64, 3, 3, 1, 1)), (-1, 2, (2, 32, 13, 13, 64, 1, 1, 1, 0)), (70, 0, (20, 512, 1, 1, 64, 1, 1, 1, 0))])
def test_split_kernels_left_alone_without_their_scratch_are_refused_with_their_need(m, tile, flags, shape):
    N, C, H, W, K, R, S, stride, pad = shape
    d = m.conv_desc(N, C, H, W, K, R, S, stride, pad, 0, m.OWT_BIAS)
    refused = 0
    for split in (1, 2):
        for p in range(3):
            m.owt_test_force_variant(tile, split, flags)
            try:
                name, bound = m.owt_conv_plan_describe(d, p), m.owt_conv_workspace_bytes(d, p)
                # those that need none: the filter gradients and the shard's forward pass unsplit, the shard's backward pass
                if name.startswith("xconv") or (name.startswith(("xfilter", "xgather", "xfc fwd")) and split == 2):
                    with pytest.raises(m.OwtError) as ei:
                        if p == 0:
                            m.owt_conv_fwd(d, 256, 512, 768, 1024, None, 0)
                        elif p == 1:
                            m.owt_conv_bwd_data(d, 256, None, 512, 1024, None, 0)
                        else:
                            m.owt_conv_bwd_filter(d, 256, 512, None, 1.0, 0.0, 1024, 768, None, 0)
                    assert ei.value.status == m.OWT_EWORKSPACE, str(ei.value)
                    need = int(str(ei.value).split("need ")[1].split()[0])
                    assert 0 < need <= bound, str(ei.value)
                    refused += 1
            finally:
                m.owt_test_force_variant(-1, 0, 0)
    assert refused


def fastest(call, rounds=20, calls=100):
    best = float("inf")
    for _ in range(rounds):
        t = time.perf_counter()
        for _ in range(calls):
            call()
        best = min(best, (time.perf_counter() - t) / calls)
    return best


def test_calls_with_little_scratch_plan_once(m):
    # what such a call runs is remembered, as for any other call: one that is refused (the fp32 kernel that it falls to splits
    # its reduction and needs more than 4 KB, so no launch comes into it) costs about what a query of the plan costs (1-2 us),
    # not a listing of the candidates (8-22 us)
    for shape in ((1, 64, 56, 56, 64, 3, 3, 1, 1), (16, 128, 56, 56, 128, 3, 3, 1, 1), (128, 64, 27, 27, 192, 5, 5, 1, 2)):
        N, C, H, W, K, R, S, stride, pad = shape
        d, text = m.conv_desc(N, C, H, W, K, R, S, stride, pad, 0, m.OWT_BIAS), ctypes.create_string_buffer(256)

        def call(nbytes=4096):
            return m._lib.owt_conv_bwd_filter(ctypes.byref(d), 256, 512, None, 1.0, 0.0, 1024, 768, 4096, nbytes, 0)

        def need(nbytes):
            m.owt_test_force_variant(-1, 0, m.OWT_FORCE_NO_BF16_MFMA)
            try:
                assert "splitk1 " not in plan(m, shape, 2), shape
            finally:
                m.owt_test_force_variant(-1, 0, 0)
            assert call(nbytes) == m.OWT_EWORKSPACE
            return int(m.owt_last_error().split("need ")[1].split()[0])

        full = plan(m, shape, 2)
        first = need(4096)
        assert fastest(call) < 2 * fastest(lambda: m._lib.owt_conv_plan_describe(ctypes.byref(d), 2, text, 256)) + 1e-6
        # the size still decides, whatever was asked before
        assert need(16) == first and need(4096) == first and plan(m, shape, 2) == full


# scratch in MB that the fp32 kernels alone ask for, and the most that may be asked for with the split-operand kernels among
# the candidates: their split filters, and partial sums only of splits that the model puts within twice its choice
@pytest.mark.parametrize("shape,p,alone,most", [((128, 3, 224, 224, 64, 11, 11, 4, 2), 0, 0.1, 0.4), ((1, 64, 56, 56, 64, 3, 3, 1, 1), 2, 5.9, 48.0),
                                                ((16, 256, 14, 14, 256, 1, 1, 1, 0), 0, 12.9, 20.0), ((2, 512, 7, 7, 512, 3, 3, 1, 1), 2, 18.9, 19.0),
                                                ((7, 64, 1024, 1100, 64, 3, 3, 1, 1), 0, 0.0, 0.0), ((128, 64, 27, 27, 192, 5, 5, 1, 2), 0, 143.3, 146.0)])
def test_workspace_bounds(m, shape, p, alone, most):
    N, C, H, W, K, R, S, stride, pad = shape
    d = m.conv_desc(N, C, H, W, K, R, S, stride, pad, 0, m.OWT_BIAS)
    bound = m.owt_conv_workspace_bytes(d, p)
    print(shape, p, bound)
    assert bound <= most * 1e6
    m.owt_test_force_variant(-1, 0, m.OWT_FORCE_NO_BF16_MFMA)
    try:
        assert m.owt_conv_workspace_bytes(d, p) <= alone * 1e6 + 1e5
    finally:
        m.owt_test_force_variant(-1, 0, 0)


# bf16 layers whose kernels differ in kind, where one was timed well ahead of another: N, C, H, W, K, R, S, stride, pad, pass, the call
# masks dy, the faster kernel, the slower one, microseconds of both
@pytest.mark.parametrize("shape,p,relu,faster,slower,us", [
    ((25, 16, 72, 75, 36, 2, 2, 2, 1), 0, True, "sconv16 ", "igemm", (13.1, 22.4)), ((2, 16, 59, 14, 56, 2, 2, 2, 1), 0, True, "sconv16 ", "igemm", (12.3, 18.1)),
    ((4, 4, 72, 46, 184, 4, 4, 3, 2), 0, True, "sconv16 ", "igemm", (13.1, 19.3)), ((52, 12, 80, 6, 120, 5, 5, 2, 0), 0, True, "igemm", "sconv16 ", (21.6, 32.5)),
    ((7, 32, 8, 12, 104, 4, 4, 2, 0), 0, True, "igemm", "sconv16x", (17.4, 23.2)), ((10, 3, 26, 107, 80, 4, 4, 2, 0), 0, True, "sconv16x", "igemm", (19.9, 25.3)),
    ((205, 96, 12, 4, 232, 3, 3, 1, 1), 1, True, "dconv16 ", "dconv16x", (28.9, 34.3)),
    ((140, 232, 13, 9, 344, 3, 3, 1, 1), 1, False, "dconv16 ", "dconv16x", (50.9, 63.7)), ((49, 200, 13, 9, 72, 5, 5, 1, 2), 0, True, "dconv16 ", "dconv16x", (27.8, 37.7)),
    ((293, 344, 35, 5, 72, 3, 3, 1, 1), 1, True, "dconv16x", "dconv16 ", (47.4, 76.0)),
    ((1, 33, 9, 62, 256, 5, 5, 1, 2), 2, False, "igemm", "ifilter16", (32.0, 42.4)), ((2, 64, 47, 48, 256, 3, 3, 1, 0), 2, False, "igemm", "ifilter16", (41.8, 49.8)),
    ((3, 130, 30, 20, 200, 5, 5, 1, 2), 2, False, "ifilter16", "igemm", (67.0, 124.0))])
def test_bf16_layers_get_the_faster_kind_of_kernel(m, shape, p, relu, faster, slower, us):
    got = plan(m, shape, p, relu, dtype=1)
    assert got.startswith(faster) and not got.startswith(slower), (got, us)


# the widest panel of the 64-pixel tile holds the loads of a masked call with an odd number of filters in scratch memory
@pytest.mark.parametrize("shape", [(13, 55, 37, 52, 11, 5, 5, 1, 2), (5, 96, 24, 53, 11, 5, 5, 1, 2), (3, 64, 34, 47, 131, 5, 5, 1, 2), (2, 47, 51, 45, 83, 5, 5, 1, 2)])
def test_wide_masked_bf16_layers_of_odd_filters_stay_off_the_tile_that_spills(m, shape):
    for tile in (-1, 93):
        m.owt_test_force_variant(tile, 0, 0)
        try:
            masked, plain = plan(m, shape, 1, True, dtype=1), plan(m, shape, 1, False, dtype=1)
        finally:
            m.owt_test_force_variant(-1, 0, 0)
        assert "waves2x1x4 panel320" not in masked, masked
        assert tile < 0 or "waves2x1x4 panel320" in plain, plain


# the shard's forward pass in one launch: long reductions of few tiles are a chain of loads there (bf16, us, split over work-groups and in one
# launch: 16 x 5632 -> 19 7.4 and 11.9, 2 x 9536 -> 430 8.0 and 13.5), and no line in the reduction's length alone parts them
@pytest.mark.parametrize("dtype,shapes,one", [
    (1, [(16, 9216, 16), (32, 8000, 64), (9, 6000, 46), (5, 6482, 41), (17, 5632, 19), (2, 9536, 430), (8, 9379, 21)], False),
    (1, [(128, 4096, 512), (128, 4500, 512), (128, 4501, 512), (61, 1792, 210), (9, 439, 46), (252, 1494, 123)], True),
    (0, [(50, 2720, 188), (16, 9216, 16), (128, 9216, 512), (8, 2614, 32)], False),
    (0, [(128, 3000, 512), (128, 3001, 512), (61, 1792, 210), (19, 632, 193), (172, 376, 44)], True)])
def test_shard_forward_in_one_launch_where_that_is_the_faster_way(m, dtype, shapes, one):
    for N, I, O in shapes:
        assert plan(m, (N, I, 1, 1, O, 1, 1, 1, 0), 0, True, dtype).startswith("xfcs" if one else "xfc "), (N, I, O)


# fp32 layers of few tiles: the 64-pixel tile where the one of 32 takes twice the work-groups for no more wavefronts (us, 64 and 32 pixels: 11.0
# and 14.0, 11.3 and 14.3, 10.7 and 13.5, 11.7 and 14.6, 14.4 and 17.3); N, C, H, W, K, R, pass, masked
@pytest.mark.parametrize("shape", [(60, 32, 14, 31, 32, 3, 1, False), (36, 13, 34, 21, 32, 3, 1, True), (16, 8, 56, 28, 32, 3, 1, False),
                                   (4, 414, 38, 16, 32, 3, 1, False), (44, 64, 41, 17, 9, 3, 0, True)])
def test_few_tiles_are_not_cut_smaller_for_a_panel_of_two_chunks(m, shape):
    N, C, H, W, K, R, p, masked = shape
    text = plan(m, (N, C, H, W, K, R, R, 1, R // 2), p, masked)
    assert text.startswith("xconvs") and "tile64x32x16" in text, text


# plans are told apart by their description without split count, grid and threads, as the benchmark groups them: a tile to a wavefront, and
# the same tile shared by four
@pytest.mark.parametrize("alone,shared,R", [(51, 53, 5), (61, 62, 3)])
def test_descriptions_tell_shared_tiles_from_others(m, alone, shared, R):
    names = []
    for tile in (alone, shared):
        m.owt_test_force_variant(tile, 0, 0)
        try:
            names.append(plan(m, (32, 64, 14, 14, 64, R, R, 1, R // 2), 2).split(" splitk")[0])
        finally:
            m.owt_test_force_variant(-1, 0, 0)
    assert names[0] != names[1] and names[1] == names[0] + " shared4", names


# bf16 filter gradients, channels in eights: the kernels that stage pixels and the two over images, where one was timed well ahead; N, C, H,
# W, K, R, the faster kernel, the slower one, microseconds of both
@pytest.mark.parametrize("shape,faster,slower,us", [
    ((46, 32, 14, 8, 32, 3), "dfilter16b ", "dfilter16 ", (14.0, 18.6)), ((3, 288, 47, 7, 480, 5), "dfilter16b ", "dfilter16 ", (34.0, 43.8)),
    ((4, 368, 10, 13, 32, 5), "dfilter16b ", "dfilter16 ", (15.7, 18.3)), ((3, 448, 19, 14, 96, 3), "dfilter16 ", "dfilter16b ", (18.9, 24.2)),
    ((909, 256, 11, 7, 64, 3), "dfilter16b ", "ifilter16b ", (51.0, 54.8)), ((340, 96, 19, 13, 160, 3), "dfilter16b ", "ifilter16b ", (56.1, 59.9)),
    ((16, 32, 9, 22, 32, 5), "ifilter16b ", "dfilter16 ", (11.0, 17.6)), ((27, 24, 18, 19, 32, 5), "ifilter16b ", "dfilter16b ", (13.0, 18.1)),
    ((9, 32, 27, 27, 144, 3), "ifilter16 ", "ifilter16b ", (14.4, 19.1)), ((349, 32, 13, 37, 320, 3), "ifilter16 ", "ifilter16b ", (61.8, 80.5))])
def test_bf16_filter_gradients_get_the_faster_kind_of_kernel(m, shape, faster, slower, us):
    N, C, H, W, K, R = shape
    got = plan(m, (N, C, H, W, K, R, R, 1, R // 2), 2, False, dtype=1)
    assert got.startswith(faster), (got, slower, us)


# masked bf16 filter gradients of one or two images, which load a mask beside every value that they gather; us over images and gathering
@pytest.mark.parametrize("shape,us", [((2, 125, 31, 12, 416, 5), (66.4, 96.9)), ((2, 324, 21, 6, 350, 5), (62.5, 84.8)), ((1, 317, 37, 43, 18, 5), (44.9, 85.6)),
                                      ((2, 47, 44, 20, 461, 3), (40.4, 62.4)), ((1, 65, 26, 28, 211, 3), (32.4, 48.7)), ((2, 96, 8, 8, 128, 5), (17.1, 24.4))])
def test_masked_bf16_filter_gradients_of_few_images_are_not_gathered(m, shape, us):
    N, C, H, W, K, R = shape
    got = plan(m, (N, C, H, W, K, R, R, 1, R // 2), 2, True, dtype=1)
    assert got.startswith("ifilter16 "), (got, us)


# fp32 passes that the kernel of few tiles and the one for layers that fill the chip are near each other on; N, C, H, W, K, R, pass, masked, the
# faster kernel, microseconds of it and of the other
@pytest.mark.parametrize("shape,faster,us", [
    ((281, 53, 10, 12, 12, 3, 0, True), "xconvs ", (19.3, 29.3)), ((127, 64, 28, 12, 8, 3, 0, True), "xconvs ", (17.1, 25.1)), ((97, 23, 40, 11, 10, 3, 0, False), "xconvs ", (12.6, 17.8)),
    ((242, 32, 12, 14, 13, 3, 0, True), "xconvs ", (11.9, 16.3)), ((58, 62, 36, 19, 10, 3, 0, True), "xconvs ", (23.4, 32.0)), ((113, 64, 12, 30, 8, 3, 0, False), "xconvs ", (19.7, 26.8)),
    ((14, 32, 35, 13, 426, 3, 1, True), "xconvs ", (33.0, 38.0)), ((32, 238, 12, 11, 115, 3, 0, False), "xconv ", (29.3, 38.6)), ((73, 42, 6, 13, 154, 3, 1, True), "xconv ", (22.3, 27.7)),
    ((116, 32, 11, 13, 212, 3, 1, False), "xconv ", (32.7, 38.4))])
def test_fp32_layers_of_some_tiles_get_the_faster_kernel(m, shape, faster, us):
    N, C, H, W, K, R, p, masked = shape
    got = plan(m, (N, C, H, W, K, R, R, 1, R // 2), p, masked)
    assert got.startswith(faster), (got, us)


# near the line between the two, us split over work-groups and in one launch: rows of whole 128-byte lines are the slower ones in one launch
@pytest.mark.parametrize("dtype,shape,one,us", [(0, (57, 2452, 19), True, (11.9, 9.1)), (1, (129, 5285, 390), True, (25.9, 12.5)), (1, (30, 8062, 46), False, (7.8, 16.3)),
                                                (0, (50, 2600, 188), True, (9.9, 9.5)), (0, (50, 2720, 188), False, (10.4, 12.0)), (1, (19, 4026, 25), True, (9.8, 7.6))])
def test_shard_forward_near_the_line(m, dtype, shape, one, us):
    N, I, O = shape
    assert plan(m, (N, I, 1, 1, O, 1, 1, 1, 0), 0, True, dtype).startswith("xfcs" if one else "xfc "), us


# fp32 strided filter gradients of few channels: what a unit of the kernels on the fp32 instruction stages is not in its clocks; us over images and
# there (N, C, H, W, K, R, S, stride, pad)
@pytest.mark.parametrize("shape,masked,us", [((176, 8, 77, 79, 320, 1, 1, 2, 0), True, (147, 766)), ((43, 8, 32, 55, 160, 1, 1, 2, 0), False, (18, 41)), ((164, 8, 25, 6, 416, 1, 3, 2, 0), False, (16, 34)),
                                             ((90, 8, 31, 79, 104, 2, 1, 3, 0), False, (20, 34)), ((235, 8, 76, 14, 504, 1, 1, 2, 0), False, (42, 273)), ((134, 16, 49, 37, 352, 1, 2, 2, 0), True, (38, 218)),
                                             ((67, 8, 11, 34, 168, 3, 1, 2, 0), False, (15, 20))])
def test_fp32_strided_filter_gradients_of_few_channels_are_taken_over_images(m, shape, masked, us):
    got = plan(m, shape, 2, masked)
    assert got.startswith("sfilterx "), (got, us)
