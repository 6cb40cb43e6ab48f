"""The ReLU mask dz = dy * [y > 0] at the values where a comparison of bits goes wrong: NaN of either sign, infinities, zeros and
subnormal numbers.  A mask only selects, so every kernel has to give, to the bit, what it gives for a mask of ones and minus ones."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, empty, force, owt, workspace  # noqa: E402

SPECIAL = {"bf16": [0x7fc0, 0x7f81, 0x7fff, 0xffc0, 0xff81, 0x7f80, 0xff80, 0x0000, 0x8000, 0x0001, 0x8001, 0x7f7f, 0x3f80, 0xbf80],
           "f32": [0x7fc00000, 0x7f800001, 0x7fffffff, 0xffc00000, 0xff800001, 0x7f800000, 0xff800000, 0, 0x80000000, 1, 0x80000001, 0x7f7fffff, 0x3f800000, 0xbf800000]}


def masks(g, shape, dt):
    """A mask of special values on the device, and one of ones and minus ones that selects the same."""
    bits = np.array(SPECIAL[dt], np.uint16 if dt == "bf16" else np.uint32)[g.integers(0, len(SPECIAL[dt]), shape)]
    value = (bits.astype(np.uint32) << 16 if dt == "bf16" else bits).view(np.float32)
    dev = torch.from_numpy(bits.view(np.int16 if dt == "bf16" else np.int32)).cuda().view(torch.bfloat16 if dt == "bf16" else torch.float32)
    return dev, torch.from_numpy(np.where(value > 0, np.float32(1), np.float32(-1))).cuda().to(dev.dtype)


def normal(g, shape, dt):
    return torch.from_numpy(g.standard_normal(shape, dtype=np.float32)).cuda().to(torch.bfloat16 if dt == "bf16" else torch.float32)


def same(a, b):
    kind = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
    return torch.equal(a.view(kind), b.view(kind))


# N, C, H, W, K, R, S, stride, pad: whole 64-channel blocks; channels in eights; odd ones; one strided first layer with filters in eights
# and one of odd geometry; 5x5; fully-connected layers
SHAPES = [(17, 64, 9, 13, 128, 3, 3, 1, 1), (4, 72, 13, 13, 136, 3, 3, 1, 1), (3, 37, 9, 14, 11, 3, 5, 1, (1, 2)), (3, 3, 36, 28, 64, 11, 11, 4, 2),
          (2, 3, 39, 39, 33, 7, 7, 4, 2), (3, 64, 27, 27, 72, 5, 5, 1, 2), (1, 35, 14, 60, 34, 5, 5, 1, 2), (9, 35, 1, 1, 33, 1, 1, 1, 0), (32, 64, 1, 1, 96, 1, 1, 1, 0)]
TILES = {"bf16": [-1] + list(range(9)) + [24] + list(range(80, 87)) + [88, 89, 90, 92, 93, 94],
         "f32": [-1] + list(range(7)) + [10, 11, 12, 16, 17, 18, 19, 22, 40, 41, 42, 43, 44, 45, 46, 50, 51, 60, 61]}
FAMILIES = {"bf16": {"igemm", "dconv16", "dconv16x", "dconv16s", "dfilter16", "sfilter16", "ifilter16", "igather16", "sfilter16x", "xfc"},
            "f32": {"igemm", "dconv", "dfilter", "sfilter", "xconv", "xconvs", "xfilter", "xgather", "sfilterx", "xfc", "fcgemm"}}


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_convolution_masks(dt):
    m, g, ran, wrong = owt(), np.random.default_rng(1700), set(), set()
    for shape in SHAPES:
        case = ConvCase(*shape, dt, True, True)
        plain = ConvCase(*shape, dt, True, False)
        x, w, dy = (normal(g, s, dt) for s in (case.shape_x, case.shape_w, case.shape_y))
        y, y1 = masks(g, case.shape_y, dt)
        xm, xm1 = masks(g, case.shape_x, dt)
        done = set()
        for tile in TILES[dt]:
            for split, flags in ((0, 0), (0, m.OWT_FORCE_ONLY_DIRECT), (2, 0)):
                with force(tile, split, flags):
                    for p in (m.OWT_PASS_BWD_DATA, m.OWT_PASS_BWD_FILTER):
                        plan = m.owt_conv_plan_describe(case.desc, p)
                        if plan in done:
                            continue
                        done.add(plan)
                        print(shape, plan)
                        sys.stdout.flush()
                        ran.add(plan.split()[0])
                        if p == m.OWT_PASS_BWD_DATA:
                            out = [empty(case.shape_x, dt) for _ in range(4)]
                            for o, mask in zip(out[:2], (y, y1)):
                                m.owt_conv_bwd_data(case.desc, dy, mask, w, o, case.ws(p))
                            for o, mask in zip(out[2:], (xm, xm1)):
                                m.owt_conv_bwd_data_relu_in(plain.desc, dy, None, w, mask, o, plain.ws(p))
                        else:
                            out = [torch.empty(s, device="cuda") for _ in range(2) for s in (case.shape_w, case.shape_w[:1])]
                            for i, mask in enumerate((y, y1)):
                                m.owt_conv_bwd_filter(case.desc, x, dy, mask, 1.0, 0.0, out[2 * i], out[2 * i + 1], case.ws(p))
                            out = [out[0], out[2], out[1], out[3]]
                        torch.cuda.synchronize()
                        if not (same(out[0], out[1]) and same(out[2], out[3])):
                            wrong.add((shape, plan))
    assert not wrong, "%d plans: %s" % (len(wrong), sorted(p for _, p in wrong))
    assert ran >= FAMILIES[dt], FAMILIES[dt] - ran


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("N,I,O", [(20, 64, 40), (7, 33, 41), (5, 48, 33), (66, 35, 64)])
def test_shard_masks(dt, N, I, O):
    m, g = owt(), np.random.default_rng(1701)
    d = m.fc_desc(N, I, O, 1, 0, m.OWT_BF16 if dt == "bf16" else m.OWT_F32, m.OWT_BIAS | m.OWT_RELU)
    x, w, dy = (normal(g, s, dt) for s in ((N, I), (O, I), (N, O)))
    for flags in (0, m.OWT_FORCE_FC_ONE_LAUNCH, m.OWT_FORCE_FC_TWO_LAUNCHES, m.OWT_FORCE_NO_BF16_MFMA):
        got = []
        for y in masks(np.random.default_rng(1702), (N, O), dt):
            out = [empty((N, I), dt), torch.empty((O, I), device="cuda"), torch.empty((O,), device="cuda")]
            with force(-1, 0, flags):
                m.owt_fc_shard_bwd(d, x, w, y, dy, 1.0, 0.0, *out, workspace(m.owt_fc_workspace_bytes(d, 1)))
            torch.cuda.synchronize()
            got.append(out)
        assert all(same(a, b) for a, b in zip(*got)), flags


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("C,win,stride", [(16, 3, 2), (5, 3, 2), (8, 2, 2)])
def test_pooling_masks(dt, C, win, stride):
    m, g, N, H = owt(), np.random.default_rng(1703), 3, 13
    P = (H - win) // stride + 1
    argmax = torch.from_numpy(g.integers(0, win * win, (N, P, P, C), dtype=np.uint8)).cuda()
    dy, got = normal(g, (N, P, P, C), dt), []
    for y in masks(g, (N, P, P, C), dt):
        dx = empty((N, H, H, C), dt)
        m.owt_maxpool_bwd_relu(N, H, H, C, win, stride, m.OWT_BF16 if dt == "bf16" else m.OWT_F32, dy, argmax, y, dx)
        torch.cuda.synchronize()
        got.append(dx)
    assert same(*got)
