"""The bf16 filter gradients over images, whose work-groups share a tile's positions between four wavefronts, against the CPU oracle.

Sizes and bounds as in test_gpu_bf16_any_channels.py: fewer positions than wavefronts, ranges that start and end inside rows and
images, ragged tiles, filters and channels in pairs and not."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, force, owt  # noqa: E402
from test_gpu_bf16_any_channels import ANY, ROWS, case_dw, check, tensors  # noqa: E402

TILES = {80: 3, 81: 3, 82: 3, 83: 3, 84: 5, 85: 5, 86: 5, 87: 0, 88: 0, 89: 0}


@pytest.mark.parametrize("split", [2, 9])
@pytest.mark.parametrize("tile", TILES)
def test_filter_gradient_shared_by_four_wavefronts(tile, split):
    m = owt()
    shapes = [s[:7] + (1, s[7]) for s in ROWS[TILES[tile]]] if TILES[tile] else ANY + [(16, 36, 1, 3, 40, 1, 1, 1, 0)]
    for i, shape in enumerate(shapes):
        N, C, H, W, K, R, S, stride, pad = shape
        x, w, b, dy, y = tensors(shape[:7] + (pad,), stride, 1300 + i)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "bf16", True, relu)
            dw0, db0 = np.full(case.shape_w, 2.0, np.float32), np.full((K,), 3.0, np.float32)
            with force(tile, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                print("case", shape, "relu", relu, plan)
                sys.stdout.flush()
                assert plan.startswith("ifilter16 " if TILES[tile] else ("sfilter16x", "igather16")), plan
                dw, db = case.bwd_filter(x, dy, y, alpha, beta, dw0, db0)
                alone, none = case.bwd_filter(x, dy, y, alpha, beta, dw0, db0, want_db=False)
            assert none is None and np.array_equal(alone, dw)
            mask = y if relu else None
            rw, rb = oracle.conv_bwd_filter(x, dy, (R, S), stride, pad, y=mask, alpha=alpha, beta=beta, dw=dw0, db=db0)
            sw, sb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), stride, pad, y=mask)
            L = N * case.P * case.Q
            check(dw, rw, sw + 2.0, L, "dw")
            check(db, rb, sb + 3.0, L, "dbias")


@pytest.mark.parametrize("tile", [t for t in TILES if TILES[t] != 5])
def test_infinities_stay_with_the_taps_that_meet_them(tile):
    shape = N, C, H, W, K, R, S, pad = (5, 33, 4, 6, 34, 3, 3, 1)
    stride = 1 if TILES[tile] else 2
    x, w, b, dy, y = tensors(shape, stride, 1390)
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "bf16", True, False)
    for at in ((0, 0, 0), (0, 1, W - 1), (4, H - 1, 0)):
        xi = x.copy()
        xi[at + (7,)] = np.inf
        with np.errstate(invalid="ignore"):
            ref = case_dw(xi, dy, R, S, pad) if stride == 1 else oracle.conv_bwd_filter(xi, dy, (R, S), stride, pad)[0]
        for split in (1, 2):
            with force(tile, split):
                dw, _ = case.bwd_filter(xi, dy, None)
            met = ~np.isfinite(ref)
            assert (~np.isfinite(dw))[met].all()
            if stride == 1:
                assert np.array_equal(np.isfinite(dw), np.isfinite(ref)) and np.array_equal(np.isnan(dw), np.isnan(ref))
