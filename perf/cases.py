"""The work whose speed counts: one worker's convolution layers, pooling, fully-connected column shards and whole
steps, each called as a program calls them (the binding's functions or ConvStack).

A case is one of four kinds:
  conv   one convolution layer, forward and backward.  "masked": the backward calls get the stored forward output and
         apply the ReLU mask themselves; otherwise dz arrives masked from its producer and backward-data applies the
         mask of the layer below, as ConvStack chains them.  "first": the layer's input is data, it has no dx.
  fc     one fully-connected column shard, forward and backward, bias + ReLU.
  pool   3x3 / stride-2 max pooling behind a ReLU, forward and backward.
  step   a whole step of the five-layer stack: fp32 with the shards, the logistic output layer and the weight update
         (one worker's training step), bf16 as the bare convolution stack.  Tuned at set-up, as bench.py does;
         the single calls run on the library's default choice of kernel, as they do for a program that does not tune.
"""
import torch

import paper_1404_5997_amd as owt
import synthetic_inputs as si
from paper_1404_5997_amd.stack import ConvStack

MOMENTUM, RATE, DECAY = 0.9, 0.01, 0.0005


def _conv(name, dtype, N, H, W, C, K, R, stride=1, pad=None, masked=False, first=False):
    return dict(name=name, kind="conv", dtype=dtype, N=N, H=H, W=W, C=C, K=K, R=R, stride=stride,
                pad=(R - 1) // 2 if pad is None else pad, masked=masked, first=first)


def listed():
    return [
        # the repository's smallest named configuration: launches and host latency are what it costs
        _conv("conv_tiny_f32", "f32", 8, 32, 32, 3, 16, 5, masked=True),
        # the five-layer stack's first layer on the per-worker batch of 128 images
        _conv("conv_first_f32", "f32", 128, 224, 224, 3, 64, 11, stride=4, pad=2, first=True),
        # its second layer: the largest share of a step
        _conv("conv_5x5_f32", "f32", 128, 27, 27, 64, 192, 5),
        # a 3x3 layer called through the plain entry points, which mask dy themselves
        _conv("conv_3x3_f32", "f32", 128, 13, 13, 192, 384, 3, masked=True),
        # a batch, a map and channel counts that divide by no tile
        _conv("conv_ragged_f32", "f32", 37, 15, 11, 100, 72, 3, masked=True),
        # bf16 storage: the second layer at a middle batch, the widest 3x3 layer at the large batch
        _conv("conv_5x5_bf16", "bf16", 256, 27, 27, 64, 192, 5),
        _conv("conv_3x3_bf16", "bf16", 1024, 13, 13, 384, 256, 3),
        # a worker's eighth of the 9216 -> 4096 layer, and the hidden shard on bf16 storage
        dict(name="fc_f32", kind="fc", dtype="f32", N=128, I=9216, O_total=4096, workers=8),
        dict(name="fc_bf16", kind="fc", dtype="bf16", N=128, I=4096, O_total=4096, workers=8),
        # the largest pooling of the bf16 stack
        dict(name="pool_bf16", kind="pool", dtype="bf16", N=512, H=55, W=55, C=64),
        # whole steps: one worker's training step in fp32, the bf16 stack at batch 1024
        dict(name="train_step_f32", kind="step", dtype="f32", N=128),
        dict(name="conv_stack_bf16", kind="step", dtype="bf16", N=1024),
    ]


def draw(rng):
    def log(lo, hi):
        return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))

    def channels(lo, hi):   # half of them whole 32-channel blocks, as networks have them
        c = log(lo, hi)
        return max(32, c // 32 * 32) if rng.random() < 0.5 else c

    kind = rng.choice(("conv", "conv", "conv", "conv", "first", "fc", "pool", "step"))
    dtype = rng.choice(("f32", "f32", "bf16"))
    if kind == "conv":
        limit = 40e9 if dtype == "f32" else 250e9
        while True:
            R = rng.choice((3, 3, 5))
            c = _conv("", dtype, log(1, 256 if dtype == "f32" else 1024), log(6, 56), log(6, 56), channels(8, 512),
                      channels(8, 512), R, masked=rng.random() < 0.5)
            if 1e7 < 2 * c["N"] * c["H"] * c["W"] * c["K"] * R * R * c["C"] < limit:
                break
    elif kind == "first":
        side = log(48, 224)
        c = _conv("", dtype, log(1, 128 if dtype == "f32" else 512), side, side, 3, rng.choice((32, 48, 64, 96)),
                  rng.choice((7, 11, 11)), stride=4, pad=2, first=True)
    elif kind == "fc":
        workers = rng.choice((1, 2, 4, 8))
        c = dict(kind="fc", dtype=dtype, N=log(1, 256), I=log(64, 9216), O_total=workers * log(16, 512), workers=workers)
    elif kind == "pool":
        c = dict(kind="pool", dtype=dtype, N=log(1, 256), H=log(6, 56), W=log(6, 56), C=channels(8, 256))
    else:
        c = dict(kind="step", dtype=dtype, N=log(1, 128 if dtype == "f32" else 512))
    c.pop("name", None)
    return c


# ------------------------------------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std)


def _storage(case):
    return (torch.bfloat16, owt.OWT_BF16) if case["dtype"] == "bf16" else (torch.float32, owt.OWT_F32)


def _out_hw(case):
    return tuple((case[k] + 2 * case["pad"] - case["R"]) // case["stride"] + 1 for k in "HW")


def _inputs(case, seed):
    """Everything random of a case, in its storage type."""
    g, (t, _) = _gen(seed), _storage(case)
    if case["kind"] == "conv":
        N, H, W, C, K, R = (case[k] for k in ("N", "H", "W", "C", "K", "R"))
        P, Q = _out_hw(case)
        if case["first"]:
            x = torch.rand((N, H, W, C), generator=g, device="cuda")      # images
        else:
            x = _normal(g, (N, H, W, C)).relu_()                           # activations behind a ReLU
        v = dict(x=x.to(t), w=_normal(g, (K, R, R, C), 0.01).to(t), b=_normal(g, (K,), 0.01), dy=_normal(g, (N, P, Q, K)).to(t))
        if case["masked"]:    # the forward output that the backward calls are given
            v["y"] = _normal(g, (N, P, Q, K)).relu_().to(t)
        return v
    if case["kind"] == "fc":
        N, I, O = case["N"], case["I"], case["O_total"] // case["workers"]
        return dict(x=_normal(g, (N, I), 0.05).relu_().to(t), w=_normal(g, (O, I), 0.005).to(t), b=_normal(g, (O,), 0.005),
                    y=_normal(g, (N, O)).relu_().to(t), dy=_normal(g, (N, O)).to(t))
    if case["kind"] == "pool":
        N, H, W, C = (case[k] for k in "NHWC")
        P, Q = (H - 3) // 2 + 1, (W - 3) // 2 + 1
        return dict(x=_normal(g, (N, H, W, C)).relu_().to(t), dy=_normal(g, (N, P, Q, C)).to(t))
    N = case["N"]
    v = dict(x=torch.rand((N,) + si.STACK_INPUT_HWC, generator=g, device="cuda").to(t), w=[], b=[])
    C = si.STACK_INPUT_HWC[2]
    for spec in si.STACK_LAYERS:
        v["w"].append(_normal(g, (spec["K"], spec["R"], spec["R"], C), 0.01).to(t))
        v["b"].append(_normal(g, (spec["K"],), 0.01))
        C = spec["K"]
    if case["dtype"] == "f32":
        v["fw"] = [_normal(g, (f["O_local"], f["I"]), 0.005) for f in si.FC_LAYERS]
        v["fb"] = [_normal(g, (f["O_local"],), 0.005) for f in si.FC_LAYERS]
        v["peers"] = [_normal(g, (N, f["O_total"] - f["O_local"]), 0.05).relu_() for f in si.FC_LAYERS[:2]]
        v["labels"] = torch.randint(0, si.FC_LAYERS[2]["O_total"], (N,), generator=g, device="cuda", dtype=torch.int32)
    else:
        v["top"] = _normal(g, (N, 6, 6, C)).to(t)
    return v


def prepare(case, seed):
    v, (t, code) = _inputs(case, seed), _storage(case)
    like = lambda shape, dtype=t: torch.empty(shape, device="cuda", dtype=dtype)   # noqa: E731
    if case["kind"] == "conv":
        N, H, W, C, K, R = (case[k] for k in ("N", "H", "W", "C", "K", "R"))
        both = owt.OWT_BIAS | owt.OWT_RELU
        v["d"] = owt.conv_desc(N, C, H, W, K, R, R, case["stride"], case["pad"], code, both)
        v["db"] = v["d"] if case["masked"] else owt.conv_desc(N, C, H, W, K, R, R, case["stride"], case["pad"], code, owt.OWT_BIAS)
        v["ws"] = like((max([16] + [owt.owt_conv_workspace_bytes(v["d"], p) for p in range(3)]),), torch.uint8)
        v["out"] = dict(y=like((N,) + _out_hw(case) + (K,)), dw=like((K, R, R, C), torch.float32), dbias=like((K,), torch.float32))
        if not case["first"]:
            v["out"]["dx"] = like((N, H, W, C))
    elif case["kind"] == "fc":
        N, I, O = case["N"], case["I"], case["O_total"] // case["workers"]
        v["d"] = owt.fc_desc(N, I, case["O_total"], case["workers"], 0, code, owt.OWT_BIAS | owt.OWT_RELU)
        v["ws"] = like((max([16] + [owt.owt_fc_workspace_bytes(v["d"], p) for p in range(2)]),), torch.uint8)
        v["out"] = dict(y=like((N, O)), dx=like((N, I)), dw=like((O, I), torch.float32), dbias=like((O,), torch.float32))
    elif case["kind"] == "pool":
        N, H, W, C = (case[k] for k in "NHWC")
        P, Q = (H - 3) // 2 + 1, (W - 3) // 2 + 1
        v["code"] = code
        v["out"] = dict(y=like((N, P, Q, C)), argmax=like((N, P, Q, C), torch.uint8), dx=like((N, H, W, C)))
    else:
        fc = si.FC_LAYERS if case["dtype"] == "f32" else None
        st = ConvStack(case["N"], si.STACK_LAYERS, si.STACK_INPUT_HWC, (si.POOL_WIN, si.POOL_STRIDE), case["dtype"], fc, si.FC_WORKERS)
        st.x.copy_(v["x"])
        for e, w, b in zip(st.L + st.F, v["w"] + v.get("fw", []), v["b"] + v.get("fb", [])):
            e["w32"].copy_(w)
            e["w"].copy_(w)
            e["b"].copy_(b)
        if fc:
            for i, peer in enumerate(v["peers"]):
                st.F[i + 1]["x"][:, st.F[i]["O"]:].copy_(peer)
            st.set_labels(v["labels"])
        else:
            st.top_grad().copy_(v["top"])
        st.autotune()
        return dict(kind="step", st=st, train=bool(fc))
    v["kind"], v["case"] = case["kind"], case
    return v


def run(s):
    if s["kind"] == "step":
        st = s["st"]
        st.step()
        if s["train"]:
            st.update(MOMENTUM, RATE, DECAY)
            return dict(loss=st.loss, logits=st.F[-1]["y"], grads=st.grads, params=st.params, vel=st.vel)
        return dict(features=st.L[-1]["a"], grads=st.grads)
    o = s["out"]
    if s["kind"] == "conv":
        y = s.get("y")
        owt.owt_conv_fwd(s["d"], s["x"], s["w"], s["b"], o["y"], s["ws"])
        owt.owt_conv_bwd_filter(s["db"], s["x"], s["dy"], y, 1.0 / s["case"]["N"], 0.0, o["dw"], o["dbias"], s["ws"])
        if not s["case"]["first"]:
            if y is not None:
                owt.owt_conv_bwd_data(s["db"], s["dy"], y, s["w"], o["dx"], s["ws"])
            else:
                owt.owt_conv_bwd_data_relu_in(s["db"], s["dy"], None, s["w"], s["x"], o["dx"], s["ws"])
    elif s["kind"] == "fc":
        owt.owt_fc_shard_fwd(s["d"], s["x"], s["w"], s["b"], o["y"], s["ws"])
        owt.owt_fc_shard_bwd(s["d"], s["x"], s["w"], s["y"], s["dy"], 1.0 / s["case"]["N"], 0.0, o["dx"], o["dw"], o["dbias"], s["ws"])
    else:
        c = s["case"]
        geom = (c["N"], c["H"], c["W"], c["C"], 3, 2, s["code"])
        owt.owt_maxpool_fwd(*geom, s["x"], o["y"], o["argmax"])
        owt.owt_maxpool_bwd_relu(*geom, s["dy"], o["argmax"], o["y"], o["dx"])
    return o


# ------------------------------------------------------------------------------------------------ yardsticks

def _layers(N):
    H, W, C = si.STACK_INPUT_HWC
    for i, spec in enumerate(si.STACK_LAYERS):
        P, Q = ((v + 2 * spec["pad"] - spec["R"]) // spec["stride"] + 1 for v in (H, W))
        yield i, spec, (N * H * W * C, spec["K"] * spec["R"] ** 2 * C, N * P * Q * spec["K"], 2 * N * P * Q * spec["K"] * spec["R"] ** 2 * C)
        H, W, C = P, Q, spec["K"]
        if spec["pool"]:
            H, W = (H - 3) // 2 + 1, (W - 3) // 2 + 1


def work(case):
    """Each tensor a call is given read once, each it fills written once; 2 operations per multiply-accumulate of the
    dense definition, taps on the padding counted."""
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "conv":
        P, Q = _out_hw(case)
        x, y, w = (case["N"] * case["H"] * case["W"] * case["C"], case["N"] * P * Q * case["K"], case["K"] * case["R"] ** 2 * case["C"])
        passes = 2 if case["first"] else 3
        nbytes = e * (x + w + y) + e * (x + y * (2 if case["masked"] else 1)) + 4 * w + 8 * case["K"]
        if not case["first"]:
            nbytes += e * (2 * y + w + x if case["masked"] else y + w + 2 * x)
        return dict(bytes=nbytes, flops=passes * 2 * w * case["N"] * P * Q)
    if case["kind"] == "fc":
        N, I, O = case["N"], case["I"], case["O_total"] // case["workers"]
        return dict(bytes=e * (N * I + O * I + N * O) + e * (N * I + O * I + 2 * N * O + N * I) + 4 * O * I + 8 * O, flops=6 * N * I * O)
    if case["kind"] == "pool":
        big = case["N"] * case["H"] * case["W"] * case["C"]
        small = case["N"] * ((case["H"] - 3) // 2 + 1) * ((case["W"] - 3) // 2 + 1) * case["C"]
        return dict(bytes=e * big + (e + 1) * small + (2 * e + 1) * small + e * big, flops=0)
    nbytes = flops = params = 0
    for i, spec, (x, w, y, f) in _layers(case["N"]):
        passes = 3 if i else 2
        nbytes += e * (x + w + y) + e * (x + y) + 4 * w + (e * (y + w + x) if i else 0)
        if spec["pool"]:
            nbytes += e * (2 * y + 3 * (y // 4)) + 2 * (y // 4)
        flops += passes * f
        params += w + spec["K"]
    if case["dtype"] == "f32":
        for f in si.FC_LAYERS:
            N, I, O = case["N"], f["I"], f["O_local"]
            nbytes += 4 * (3 * N * I + 3 * O * I + 4 * N * O)
            flops += 6 * N * I * O
            params += O * I + O
        nbytes += 20 * params
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """Four times what a call differs by from the 64-bit result or, where bf16 results are rounded when stored, from
    the same call with its sums split differently."""
    if case["kind"] == "pool":
        return dict(rel=1e-6, max=1e-5) if case["dtype"] == "f32" else dict(rel=4e-3, max=4e-2)
    if case["kind"] == "step":
        return dict(rel=2e-3, max=0.5) if case["dtype"] == "f32" else dict(rel=2e-2, max=0.9)
    return dict(rel=1e-5, max=1e-4) if case["dtype"] == "f32" else dict(rel=4e-3, max=4e-2)


# ------------------------------------------------------------------------------------------------ 64-bit results

def _taps(case_hw, R, stride, pad, P, Q):
    """The rows and columns of the padded image that each filter tap meets."""
    for r in range(R):
        for s in range(R):
            yield r, s, slice(r, r + (P - 1) * stride + 1, stride), slice(s, s + (Q - 1) * stride + 1, stride)


def _pad64(x, pad):
    N, H, W, C = x.shape
    out = torch.zeros((N, H + 2 * pad, W + 2 * pad, C), device=x.device, dtype=torch.float64)
    out[:, pad:pad + H, pad:pad + W] = x
    return out


def _conv64(x, w, b, stride, pad):
    (N, H, W, C), (K, R) = x.shape, w.shape[:2]
    P, Q = ((v + 2 * pad - R) // stride + 1 for v in (H, W))
    xp, y = _pad64(x, pad), b.double().repeat(N * P * Q, 1)
    for r, s, rows, cols in _taps((H, W), R, stride, pad, P, Q):
        y += xp[:, rows, cols].reshape(-1, C) @ w[:, r, s].double().t().contiguous()
    return y.view(N, P, Q, K)


def _pool64(x):
    N, H, W, C = x.shape
    P, Q = (H - 3) // 2 + 1, (W - 3) // 2 + 1
    best = torch.full((N, P, Q, C), -torch.inf, device=x.device, dtype=torch.float64)
    where = torch.zeros((N, P, Q, C), device=x.device, dtype=torch.uint8)
    for r, s, rows, cols in _taps((H, W), 3, 2, 0, P, Q):
        v = x[:, rows, cols].double()
        more = v > best
        best = torch.where(more, v, best)
        where = where.masked_fill(more, 3 * r + s)
    return best, where


def exact(case, seed):
    v = _inputs(case, seed)
    if case["kind"] == "conv":
        N, H, W, C, R, pad = (case[k] for k in ("N", "H", "W", "C", "R", "pad"))
        P, Q = _out_hw(case)
        out = dict(y=_conv64(v["x"], v["w"], v["b"], case["stride"], pad).relu_())
        dz = v["dy"].double().view(-1, case["K"])
        if case["masked"]:
            dz = dz * (v["y"].view(-1, case["K"]) > 0)
        xp = _pad64(v["x"], pad)
        dw = torch.zeros(v["w"].shape, device="cuda", dtype=torch.float64)
        dxp = None if case["first"] else torch.zeros_like(xp)
        dzt = dz.t().contiguous()
        for r, s, rows, cols in _taps((H, W), R, case["stride"], pad, P, Q):
            dw[:, r, s] = dzt @ xp[:, rows, cols].reshape(-1, C)
            if dxp is not None:
                dxp[:, rows, cols] += (dz @ v["w"][:, r, s].double()).view(N, P, Q, C)
        out.update(dw=dw / N, dbias=dz.sum(0) / N)
        if dxp is not None:
            dx = dxp[:, pad:pad + H, pad:pad + W]
            out["dx"] = (dx if case["masked"] else dx * (v["x"] > 0)).contiguous()
        return out
    if case["kind"] == "fc":
        x, w = v["x"].double(), v["w"].double()
        dz = v["dy"].double() * (v["y"] > 0)
        return dict(y=(x @ w.t().contiguous() + v["b"].double()).relu_(), dx=dz @ w, dw=dz.t().contiguous() @ x / case["N"],
                    dbias=dz.sum(0) / case["N"])
    if case["kind"] == "pool":
        y, where = _pool64(v["x"])
        dx = torch.zeros(v["x"].shape, device="cuda", dtype=torch.float64)
        dy = v["dy"].double() * (y > 0)
        for r, s, rows, cols in _taps((case["H"], case["W"]), 3, 2, 0, *y.shape[1:3]):
            dx[:, rows, cols] += dy * (where == 3 * r + s)
        return dict(y=y, argmax=where, dx=dx)
    # The forward outputs.  The gradients of a free-running step have no 64-bit value to be held against: an
    # activation at the edge of a ReLU or a window with two near-equal maxima sends its gradient one way or the other.
    cur = v["x"].double()
    for spec, w, b in zip(si.STACK_LAYERS, v["w"], v["b"]):
        cur = torch.cat([_conv64(part, w, b, spec["stride"], spec["pad"]).relu_() for part in cur.split(128)])
        if spec["pool"]:
            cur = _pool64(cur)[0]
    if case["dtype"] == "bf16":
        return dict(features=cur, grads=None)
    cur = cur.reshape(case["N"], -1)
    for i, (w, b) in enumerate(zip(v["fw"], v["fb"])):
        if i:
            cur = torch.cat([cur, v["peers"][i - 1].double()], 1)
        cur = cur @ w.double().t().contiguous() + b.double()
        if si.FC_LAYERS[i]["relu"]:
            cur = cur.relu_()
    hit = torch.arange(cur.shape[1], device="cuda")[None] == v["labels"][:, None]
    loss = (torch.nn.functional.softplus(cur) - cur * hit).sum(1)
    return dict(loss=loss, logits=cur, grads=None, params=None, vel=None)
