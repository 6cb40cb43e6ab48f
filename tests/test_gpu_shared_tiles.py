"""The fp32 filter gradients whose work-groups share a tile's positions between four wavefronts, against the CPU oracle.

Sizes: fewer positions than wavefronts, a part of them empty, ranges that start and end inside rows and images, ragged tiles.  Bounds
as in test_gpu_split.py."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import ConvCase, force, owt  # noqa: E402
from test_gpu_split import FILTER_SHAPES, STRIDED, check, conv64, strided_tensors, tensors  # noqa: E402

ANY = STRIDED + [(17, 5, 6, 7, 70, 3, 3, 1, 1), (1, 1, 8, 8, 1, 3, 3, 1, 1), (5, 36, 4, 4, 40, 1, 1, 1, 0), (3, 4, 5, 5, 4, 3, 3, 1, 2), (2, 7, 1, 2, 5, 1, 1, 1, 0)]


def shapes(tile):
    return [s[:7] + (1, s[7]) for s in FILTER_SHAPES[tile - 52]] if tile < 60 else ANY


@pytest.mark.parametrize("tile,split", [(52, 1), (52, 2), (52, 9), (53, 1), (53, 3), (53, 16), (62, 1), (62, 3), (63, 1), (63, 7)])
def test_filter_gradient_shared_by_four_wavefronts(tile, split):
    m = owt()
    for i, shape in enumerate(shapes(tile)):
        N, C, H, W, K, R, S, stride, pad = shape
        x, w, b, dy, y = tensors(shape[:7] + (pad,), 1900 + i) if tile < 60 else strided_tensors(shape, 1900 + i)
        for relu, alpha, beta in ((False, 1.0, 0.0), (True, 0.5, -0.25)):
            case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", True, relu)
            g = np.random.default_rng(1920 + i)
            dw0 = g.standard_normal(case.shape_w, dtype=np.float32) if beta else None
            db0 = g.standard_normal((K,), dtype=np.float32) if beta else None
            with force(tile, split):
                plan = m.owt_conv_plan_describe(case.desc, 2)
                print("case", shape, "relu", relu, plan)
                sys.stdout.flush()
                assert plan.startswith(("xfilter", "xgather", "sfilterx")), plan
                dw, db = case.bwd_filter(x, dy, y if relu else None, alpha, beta, dw0, db0)
                alone, none = case.bwd_filter(x, dy, y if relu else None, alpha, beta, dw0, db0, want_db=False)
            assert none is None and np.array_equal(alone, dw)
            mask = y if relu else None
            ref, rdb = oracle.conv_bwd_filter(x, dy, (R, S), stride, pad, y=mask, alpha=alpha, beta=beta, dw=dw0, db=db0)
            size, sdb = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), (R, S), stride, pad, y=mask, alpha=alpha, beta=abs(beta),
                                               dw=None if dw0 is None else np.abs(dw0), db=None if db0 is None else np.abs(db0))
            L = N * case.P * case.Q
            check(dw, ref, size, L, "dw")
            check(db, rdb, sdb, L, "db", norm_too=False)


@pytest.mark.parametrize("tile,shape", [(52, (18, 40, 6, 7, 70, 3, 3, 1, 1)), (53, (18, 40, 6, 7, 33, 5, 5, 1, 2)), (62, (18, 3, 23, 20, 30, 7, 7, 4, 2)), (63, (18, 3, 23, 20, 30, 7, 7, 4, 2))])
def test_ends_of_the_range_and_what_is_not_finite(tile, shape):
    N, C, H, W, K, R, S, stride, pad = shape
    case = ConvCase(N, C, H, W, K, R, S, stride, pad, "f32", False, False)

    def want(x, dy):
        ref = np.zeros(case.shape_w)
        with np.errstate(all="ignore"):
            for r, s, xs in conv64(x, np.zeros(case.shape_w), stride, pad, case.P, case.Q)[1]:
                ref[:, r, s] = dy.reshape(-1, K).astype(np.float64).T @ xs.reshape(-1, C)
        return ref
    # operands so small that their low parts leave bf16's range, and so large that a product of high parts would be infinite: each
    # wavefront looks at its own sums, so one of them may start over scaled and another not
    for a, b in ((2.0 ** -118, 2.0 ** 20), (2.0 ** 106, 2.0 ** -100)):
        g = np.random.default_rng(1950)
        x, dy = (g.standard_normal(case.shape_x) * a).astype(np.float32), (g.standard_normal(case.shape_y) * b).astype(np.float32)
        ref = want(x, dy)
        for split in (1, 3):
            with force(tile, split):
                dw, _ = case.bwd_filter(x, dy, None, want_db=False)
            err = np.linalg.norm(dw - ref) / np.linalg.norm(ref)
            print("  tile", tile, a, b, split, err)
            sys.stdout.flush()
            assert err < 1e-6                          # every bit of an operand counts; bits lost at the ends show as 1e-5 and more
    g = np.random.default_rng(1960)
    x, dy = g.standard_normal(case.shape_x).astype(np.float32), g.standard_normal(case.shape_y).astype(np.float32)
    x[0, 1, 1, 2], x[N - 1, 2, 3, 0] = np.inf, np.nan
    ref = want(x, dy)
    for split in (1, 2):
        with force(tile, split):
            dw, _ = case.bwd_filter(x, dy, None, want_db=False)
        met = ~np.isfinite(ref)
        assert met.any() and (~np.isfinite(dw))[met].all()
        if stride > 1:                                 # (a tap that no window position takes to them stays finite)
            assert np.isfinite(dw[~met]).all() and np.allclose(dw[~met], ref[~met], rtol=1e-4, atol=1e-3)
