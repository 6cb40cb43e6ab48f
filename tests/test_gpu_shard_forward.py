"""The dense shard's forward pass in one launch (16 x 16 tiles), against the CPU oracle.

Bounds as in test_gpu_split.py (fp32) and test_gpu_bf16_any_channels.py (bf16)."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import empty, force, owt, to_dev, to_host, workspace  # noqa: E402
import test_gpu_bf16_any_channels as b16  # noqa: E402
import test_gpu_split as f32  # noqa: E402


def run(m, x, w, b, dt, flags, workers=1):
    (N, I), O = x.shape, w.shape[0]
    d = m.fc_desc(N, I, O * workers, workers, 0, m.OWT_BF16 if dt == "bf16" else m.OWT_F32, flags)
    c = m.conv_desc(N, I, 1, 1, O, 1, 1, 1, 0, m.OWT_BF16 if dt == "bf16" else m.OWT_F32, flags)
    with force(71, 0):
        assert m.owt_conv_plan_describe(c, 0).startswith("xfcs"), m.owt_conv_plan_describe(c, 0)
        y, ws = empty((N, O), dt), workspace(m.owt_fc_workspace_bytes(d, 0))
        m.owt_fc_shard_fwd(d, to_dev(x, dt), to_dev(w, dt), to_dev(b), y, ws)
        torch.cuda.synchronize()
    return to_host(y)


# N, I, O: one tile less and more than full, one value, reductions shorter than a step, than the wavefronts' first steps, ending one value
# into a step and one before its end, odd ones (bf16 rows at any 2 bytes), more tiles than XCDs deal out evenly
SHAPES = [(1, 1, 1), (16, 32, 16), (17, 31, 15), (3, 64, 33), (33, 65, 100), (5, 511, 17), (128, 513, 40), (130, 1025, 70), (7, 2111, 260), (64, 4096, 16)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_shard_forward_in_one_launch(dt):
    m = owt()
    for i, (N, I, O) in enumerate(SHAPES):
        g = np.random.default_rng(2100 + i)
        x, w, b = (g.standard_normal(s, dtype=np.float32) for s in ((N, I), (O, I), (O,)))
        if dt == "bf16":
            x, w = oracle.round_bf16(x), oracle.round_bf16(w)
        ref = x.astype(np.float64) @ w.T.astype(np.float64)
        size = np.abs(x).astype(np.float64) @ np.abs(w).T.astype(np.float64)
        for flags in (0, m.OWT_BIAS | m.OWT_RELU):
            print("case", dt, (N, I, O), flags)
            sys.stdout.flush()
            want, sz = (ref, size) if not flags else (np.maximum(ref + b, 0.0), size + np.abs(b))
            got = run(m, x, w, b if flags else None, dt, flags)
            if dt == "bf16":
                b16.check(got, want, sz, I, "y", stored=2.0 ** -8)
            else:
                f32.check(got, want.astype(np.float32), sz.astype(np.float32), I, "y", norm_too=N * O > 16)     # (one value, and it zero, has no norm)


def test_what_is_not_finite_stays_in_its_row_and_column():
    m = owt()
    for dt in ("f32", "bf16"):
        for I in (70, 201):
            g = np.random.default_rng(2150)
            x, w = (g.standard_normal(s, dtype=np.float32) for s in ((40, I), (50, I)))
            if dt == "bf16":
                x, w = oracle.round_bf16(x), oracle.round_bf16(w)
            x[7, I - 1], x[20, 3], w[33, 0] = np.inf, np.nan, np.float32(3e38)
            with np.errstate(all="ignore"):
                ref = (x.astype(np.float64) @ w.T.astype(np.float64)).astype(np.float32)
            got = run(m, x, w, None, dt, 0)
            bad = ~np.isfinite(ref)
            assert (np.isfinite(got) == ~bad).all(), (dt, I)
            assert (np.isnan(got) == np.isnan(ref)).all(), (dt, I)
            assert np.allclose(got[~bad], ref[~bad], rtol=1e-2 if dt == "bf16" else 1e-4, atol=1e-3), (dt, I)


@pytest.mark.parametrize("a,b", [(2.0 ** -118, 2.0 ** 20), (2.0 ** 106, 2.0 ** -100), (2.0 ** 50, 2.0 ** 50)])
def test_ends_of_the_fp32_range(a, b):
    m = owt()
    g = np.random.default_rng(2160)
    x, w = (g.standard_normal((40, 300)) * a).astype(np.float32), (g.standard_normal((50, 300)) * b).astype(np.float32)
    f32.check_ends(run(m, x, w, None, "f32", 0), x.astype(np.float64) @ w.T.astype(np.float64), 300, "y")


# the longest reductions that it is chosen for, and those that it was chosen for once: rows that start at 4 and at 16 bytes, and at any 2 in bf16
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_long_reductions(dt):
    m = owt()
    for i, (N, I, O) in enumerate([(9, 6000, 46), (16, 9216, 16), (128, 4096, 512), (128, 7680, 512), (5, 6483, 41), (33, 12001, 17)]):
        g = np.random.default_rng(2180 + i)
        x, w = (g.standard_normal(s, dtype=np.float32) for s in ((N, I), (O, I)))
        if dt == "bf16":
            x, w = oracle.round_bf16(x), oracle.round_bf16(w)
        print("case", dt, (N, I, O))
        sys.stdout.flush()
        got, want = run(m, x, w, None, dt, 0), x.astype(np.float64) @ w.T.astype(np.float64)
        size = np.abs(x).astype(np.float64) @ np.abs(w).T.astype(np.float64)
        if dt == "bf16":
            b16.check(got, want, size, I, "y", stored=2.0 ** -8)
        else:
            f32.check(got, want.astype(np.float32), size.astype(np.float32), I, "y")
