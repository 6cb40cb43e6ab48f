"""Which calls are refused for their scratch, without a device: one that is accepted fails at its launch instead.

The sizes are those below which each call has been refused since sizes were handed out; kernels and prices that came later neither
refuse a call nor take one that was refused (its tensors may be as small as the caller's mistake made them)."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
import paper_1404_5997_amd as owt  # noqa: E402

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="the pointers are made up")

CASES = [
    (1, (6, 120, 18, 16, 32, 3, 3, 1, 1, False), 0, [(0, True), (65536, True), (119808, False)]),
    (1, (6, 120, 18, 16, 32, 3, 3, 1, 1, False), 1, [(0, True), (68864, True), (69120, False)]),
    (1, (6, 120, 18, 16, 32, 3, 3, 1, 1, False), 2, [(0, True), (1048576, True), (1660416, False)]),
    (1, (29, 75, 13, 13, 96, 3, 3, 1, 1, True), 0, [(0, True), (65536, True), (1048576, False)]),
    (1, (29, 75, 13, 13, 96, 3, 3, 1, 1, True), 1, [(0, True), (65536, True), (1048576, False)]),
    (1, (29, 75, 13, 13, 96, 3, 3, 1, 1, True), 2, [(0, True), (65536, True), (1048576, False)]),
    (1, (45, 79, 9, 7, 384, 3, 3, 1, 1, False), 2, [(0, True), (1048576, True), (4194304, False)]),
    (1, (22, 255, 19, 16, 110, 3, 3, 1, 1, True), 2, [(0, True), (1048576, True), (4194304, False)]),
    (1, (7, 136, 63, 12, 322, 1, 1, 2, 0, True), 1, [(0, True), (11515136, True), (11515392, False)]),
    (1, (7, 136, 63, 12, 322, 1, 1, 2, 0, True), 2, [(0, True), (65536, True), (1048576, False)]),
    (1, (3, 167, 6, 25, 18, 7, 7, 4, 3, True), 0, [(0, True), (386816, True), (387072, False)]),
    (1, (16, 251, 3, 6, 12, 3, 3, 4, 1, False), 0, [(0, True), (44288, True), (44544, False)]),
    (1, (3, 110, 44, 23, 83, 1, 1, 2, 0, False), 2, [(0, True), (65536, True), (244160, False)]),
    (1, (119, 149, 13, 12, 8, 3, 3, 2, 0, False), 2, [(0, True), (65536, True), (322112, False)]),
    (1, (2, 8, 56, 62, 347, 3, 3, 2, 0, True), 2, [(0, True), (1048576, True), (2571136, False)]),
    (1, (3, 306, 7, 25, 8, 4, 4, 2, 0, False), 1, [(0, True), (1285120, True), (1285376, False)]),
    (0, (1, 312, 26, 6, 450, 3, 3, 1, 1, False), 0, [(0, True), (1048576, True), (1456928, False)]),
    (0, (1, 312, 26, 6, 450, 3, 3, 1, 1, False), 1, [(0, True), (8203776, True), (10938112, False)]),
    (0, (1, 312, 26, 6, 450, 3, 3, 1, 1, False), 2, [(0, True), (7584320, True), (15168640, False)]),
    (0, (62, 37, 15, 26, 202, 3, 3, 1, 1, True), 1, [(0, True), (65536, True), (1048576, False)]),
    (0, (62, 37, 15, 26, 202, 3, 3, 1, 1, True), 2, [(0, True), (1048576, True), (4194304, False)]),
    (0, (105, 32, 14, 31, 272, 5, 5, 1, 2, False), 2, [(0, True), (4194304, True), (16777216, False)]),
    (0, (12, 24, 32, 11, 32, 3, 3, 1, 1, True), 2, [(0, True), (409728, True), (819456, False)]),
    (0, (4, 416, 31, 53, 448, 3, 3, 1, 1, True), 0, [(0, True), (4194304, True), (16777216, False)]),
    (0, (7, 136, 63, 12, 322, 1, 1, 2, 0, True), 1, [(0, True), (11515136, True), (11515392, False)]),
    (0, (7, 136, 63, 12, 322, 1, 1, 2, 0, True), 2, [(0, True), (65536, True), (1048576, False)]),
    (0, (3, 167, 6, 25, 18, 7, 7, 4, 3, True), 0, [(0, True), (386816, True), (387072, False)]),
    (0, (16, 251, 3, 6, 12, 3, 3, 4, 1, False), 0, [(0, True), (44288, True), (44544, False)]),
    (0, (3, 110, 44, 23, 83, 1, 1, 2, 0, False), 2, [(0, True), (65536, True), (244160, False)]),
    (0, (119, 149, 13, 12, 8, 3, 3, 2, 0, False), 2, [(0, True), (257664, True), (515328, False)]),
    (0, (2, 8, 56, 62, 347, 3, 3, 2, 0, True), 2, [(0, True), (2051840, True), (4103680, False)]),
    (0, (3, 306, 7, 25, 8, 4, 4, 2, 0, False), 1, [(0, True), (1285120, True), (1285376, False)]),
    (1, (16, 192, 13, 13, 384, 3, 3, 1, 1, False), 2, [(0, True), (19254144, True), (38508288, False)]),
    (0, (16, 192, 13, 13, 384, 3, 3, 1, 1, False), 2, [(0, True), (4194304, True), (9627072, False)]),
    (0, (128, 9216, 512), "shard", [(0, True), (1048576, True), (3801088, False)]),
    (1, (128, 4096, 512), "shard", [(0, True), (65536, True), (1048576, False)]),
    (0, (128, 4096, 125), "shard", [(0, True), (65536, True), (512000, False)]),
    (1, (5, 6482, 41), "shard", [(0, True), (16, True), (4096, False)]),
]


def refused(dtype, shape, pass_, size):
    at, lib, none = (lambda i: ctypes.c_void_p(i << 32)), owt._lib, ctypes.c_void_p(0)
    scratch = (at(9) if size else none, ctypes.c_size_t(size), none)
    if pass_ == "shard":
        d = owt.fc_desc(*shape, 1, 0, dtype, owt.OWT_BIAS | owt.OWT_RELU)
        status = lib.owt_fc_shard_fwd(ctypes.byref(d), at(1), at(2), at(3), at(4), *scratch)
    else:
        N, C, H, W, K, R, S, stride, pad, masked = shape
        d = owt.conv_desc(N, C, H, W, K, R, S, stride, pad, dtype, 3 if masked else 1)
        call = (lib.owt_conv_fwd, lib.owt_conv_bwd_data, lib.owt_conv_bwd_filter)[pass_]
        args = (at(1), at(2), at(3), at(4)) if pass_ < 2 else (at(1), at(2), at(3), ctypes.c_float(1), ctypes.c_float(0), at(4), at(5))
        status = call(ctypes.byref(d), *args, *scratch)
    assert status != 0
    return status == owt.OWT_EWORKSPACE


@pytest.mark.parametrize("dtype,shape,pass_,refusals", CASES)
def test_calls_are_refused_for_their_scratch_as_ever(dtype, shape, pass_, refusals):
    for size, expected in refusals:
        assert refused(dtype, shape, pass_, size) == expected, size
