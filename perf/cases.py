"""What this library is timed on: training steps of whole stacks through ff_train_step, and the single operations of one
layer (forward: quantise, contraction, goodness, hand-off; backward: local gradient, weight gradient, update) as a training
loop of one's own calls them.

Sizes are those of `workloads` (the paper's MNIST-shaped and CIFAR-shaped networks, a ResNet-18-shaped and a
MobileNet-shaped stack, a large dense stack) plus odd ones of the same kinds.  Inputs are synthetic and made from the seed.
Goodness thresholds are set per layer to the median goodness at the initial weights, so that the positive and the negative
set both carry gradients, as they do while a network trains.  The rates are small enough that thousands of passes over one
batch stay in that regime (a convolution's gradient is a sum over every pixel of its map: a hundredth of the dense rate).

`exact` restates the method in 64 bits with plain torch: quantisers, contractions, goodness, look-ahead, update."""
from __future__ import annotations

import dataclasses
import math

import torch

import paper_2506_22771_amd as ff
from paper_2506_22771_amd import schedule
from workloads import Layer, bottleneck_stack, mlp, res_stack

LR = {"mlp": 1e-4, "cnn": 1e-6, "residual": 1e-6, "bottleneck": 1e-6}
SR_SEED = 2


def listed():
    return [
        # the paper's MNIST-shaped MLP at a small batch: latency of one step
        {"name": "step_mlp_small", "what": "step", "net": "mlp", "widths": "784-500-500", "batch": 64, "l2norm": False,
         "lam": 0.0, "chain": False, "data": "pixels"},
        # the wider MNIST-shaped MLP with look-ahead and normalised hand-off, an ordinary batch
        {"name": "step_mlp", "what": "step", "net": "mlp", "widths": "784-2000-2000-2000-2000", "batch": 1024,
         "l2norm": True, "lam": 0.05, "chain": False, "data": "pixels"},
        # large dense layers: the contractions at full size
        {"name": "step_mlp_large", "what": "step", "net": "mlp", "widths": "4096-4096-4096", "batch": 8192,
         "l2norm": False, "lam": 0.05, "chain": False, "data": "normal"},
        # Eq. (4) as an exact derivative through the later layers; widths and batch that are no powers of two
        {"name": "step_mlp_chain", "what": "step", "net": "mlp", "widths": "1000-1500-1500-1001", "batch": 1500,
         "l2norm": False, "lam": 0.05, "chain": True, "data": "normal"},
        # CIFAR-shaped plain CNN, 3x3 convolutions at full resolution
        {"name": "step_cnn", "what": "step", "net": "cnn", "map": 32, "channels": "3-64-128-256", "strides": "1-1-1",
         "head": 0, "batch": 256, "lam": 0.0},
        # MNIST-shaped CNN: one input channel, 28 -> 14 -> 7 pixels by stride 2, a dense head; an odd batch
        {"name": "step_cnn_28", "what": "step", "net": "cnn", "map": 28, "channels": "1-32-48-96", "strides": "1-2-2",
         "head": 500, "batch": 100, "lam": 0.05},
        # ResNet-18-shaped stack on CIFAR-shaped images
        {"name": "step_resnet", "what": "step", "net": "residual", "map": 32, "stages": "64-128-256-512", "blocks": 2,
         "batch": 256, "lam": 0.05},
        # MobileNet-V2-shaped first stages: 1x1 and depthwise convolutions
        {"name": "step_mobile", "what": "step", "net": "bottleneck", "map": 32, "stem": 32,
         "blocks": "1x16s1-6x24s1-6x24s1-6x32s2-6x32s1", "batch": 256, "lam": 0.05},
        # one dense layer forward in a loop of one's own, ragged sizes
        {"name": "dense_forward", "what": "forward", "net": "mlp", "widths": "784-1201", "batch": 1000, "l2norm": True,
         "lam": 0.0, "chain": False, "data": "pixels"},
        # one dense layer backward: both sets' gradients and the update
        {"name": "dense_backward", "what": "backward", "net": "mlp", "widths": "2000-2000", "batch": 2048,
         "l2norm": False, "lam": 0.0, "chain": False, "data": "normal"},
        # one convolution forward in the middle of a CIFAR-shaped network
        {"name": "conv_forward", "what": "forward", "net": "cnn", "map": 16, "channels": "128-256", "strides": "1",
         "head": 0, "batch": 256, "lam": 0.0},
        # one convolution backward at full resolution (two accumulators per set: the reduction exceeds int32)
        {"name": "conv_backward", "what": "backward", "net": "cnn", "map": 32, "channels": "64-128", "strides": "1",
         "head": 0, "batch": 256, "lam": 0.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = sum(_macs(c) for c in listed() if c["name"] == "step_mlp_large")
    while True:
        net = rng.choice(["mlp", "mlp", "mlp", "cnn", "cnn", "residual", "bottleneck"])
        lam = rng.choice([0.0, 0.001, 0.05])
        if net == "mlp":
            what = rng.choice(["step", "step", "step", "forward", "backward"])
            depth = rng.randint(2, 4) if what == "step" else 1
            chain = what == "step" and rng.random() < 0.25
            c = {"what": what, "net": net, "widths": "-".join(str(_log_int(rng, 50, 4096)) for _ in range(depth + 1)),
                 "batch": _log_int(rng, 16, 8192), "l2norm": not chain and rng.random() < 0.5, "lam": lam, "chain": chain,
                 "data": rng.choice(["pixels", "normal"])}
        elif net == "cnn":
            what = rng.choice(["step", "step", "forward", "backward"])
            side = rng.choice([28, 32, rng.randint(7, 32)])
            depth = rng.randint(2, 3) if what == "step" else 1
            chans = [rng.choice([1, 3]) if what == "step" else 8 * rng.randint(2, 16)]
            chans += [8 * rng.randint(2, 32) for _ in range(depth)]
            c = {"what": what, "net": net, "map": side, "channels": "-".join(map(str, chans)),
                 "strides": "-".join(str(rng.choice([1, 1, 2])) for _ in range(depth)),
                 "head": rng.choice([0, 0, 10 * rng.randint(5, 50)]) if what == "step" else 0,
                 "batch": _log_int(rng, 16, 256), "lam": lam}
        elif net == "residual":
            n = rng.randint(1, 4)
            c = {"what": "step", "net": net, "map": rng.choice([28, 32]),
                 "stages": "-".join(str((32 if rng.random() < 0.5 else 64) << i) for i in range(n)),
                 "blocks": rng.randint(1, 2), "batch": _log_int(rng, 16, 256), "lam": lam}
        else:
            blocks = "-".join("%dx%ds%d" % (rng.choice([1, 3, 6]), 8 * rng.randint(2, 5), rng.choice([1, 1, 2]))
                              for _ in range(rng.randint(1, 4)))
            c = {"what": "step", "net": net, "map": rng.choice([28, 32]), "stem": 32, "blocks": blocks,
                 "batch": _log_int(rng, 16, 256), "lam": lam}
        # no costlier than the largest listed case, in arithmetic and in activations held
        if _macs(c) <= most and sum(l.terms_per_sample for l in _layers(c)) * c["batch"] <= 240e6:
            return c


def _ints(s):
    return [int(v) for v in s.split("-")]


def _layers(c):
    if c["net"] == "mlp":
        layers = mlp(_ints(c["widths"]), c["l2norm"])
        if c["what"] != "step":   # a single layer that hands its (normalised) output on
            layers = tuple(dataclasses.replace(l, l2norm_out=int(c["l2norm"])) for l in layers)
        return layers
    if c["net"] == "cnn":
        chans, side, out = _ints(c["channels"]), c["map"], []
        for a, b, s in zip(chans, chans[1:], _ints(c["strides"])):
            out.append(Layer("conv", H=side, W=side, C_in=a, C_out=b, ksize=3, stride=s, pad=1))
            side = out[-1].H_out
        if c["head"]:
            out.append(Layer("dense", in_features=side * side * chans[-1], out_features=c["head"]))
        return tuple(out)
    if c["net"] == "residual":
        st = _ints(c["stages"])
        return res_stack(st[0], [(ch, 2 if i else 1, c["blocks"]) for i, ch in enumerate(st)], c["map"], c["map"])
    blocks = []
    for b in c["blocks"].split("-"):
        t, rest = b.split("x")
        ch, s = rest.split("s")
        blocks.append((int(t), int(ch), int(s)))
    return bottleneck_stack(c["stem"], blocks, c["map"], c["map"])


def _inputs(c, layers, seed):
    """Both data sets and the master weights, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    first, B = layers[0], c["batch"]
    n = first.in_elems_per_sample
    if c.get("data", "pixels") == "normal":
        xp = torch.randn((B, n), generator=g, device="cuda")
        xn = torch.randn((B, n), generator=g, device="cuda")
    else:   # pixel values with the label as one-hot over ten leading features (convolutions: pixels of channel 0)
        xp = torch.rand((B, n), generator=g, device="cuda")
        xn = xp.clone()
        true = torch.randint(0, 10, (B,), generator=g, device="cuda")
        wrong = (true + torch.randint(1, 10, (B,), generator=g, device="cuda")) % 10
        step = 1 if first.kind == "dense" else first.C_in
        slots = min(10, n // step)
        for x, lab in ((xp, true), (xn, wrong)):
            x[:, :slots * step:step] = torch.nn.functional.one_hot(lab, 10)[:, :slots].float()
    w = []
    for l in layers:
        bound = math.sqrt(6.0 / l.fan_in)
        w.append((torch.rand((l.N, l.K), generator=g, device="cuda") * 2 - 1) * bound)
    return xp, xn, w


def _three_digits(v):
    return float("%.3g" % v)


def prepare(case, seed):
    layers = _layers(case)
    xp, xn, w = _inputs(case, layers, seed)
    return {"step": _prepare_step, "forward": _prepare_forward, "backward": _prepare_backward}[case["what"]](case, layers, xp, xn, w)


def run(state):
    return {"step": _run_step, "forward": _run_forward, "backward": _run_backward}[state["what"]](state)


# ---- whole steps -------------------------------------------------------------------------------------------------------

def _prepare_step(case, layers, xp, xn, w):
    B, k = case["batch"], len(layers)
    st = schedule.TrainState.from_weights(layers, B, w)
    look = "chain" if case.get("chain") else "coeff"
    loss = torch.empty((k, 2), device="cuda")
    good = torch.empty((k, 2, B), device="cuda")
    net = st.net(lookahead=look)
    ws = torch.empty(net.workspace_bytes(), dtype=torch.uint8, device="cuda")
    ff.ff_train_step(net, xp, xn, 2.0, case["lam"], 0.0, SR_SEED, 0, loss, good, ws)   # rate 0: goodness at the start
    theta = [_three_digits(v) for v in good.reshape(k, -1).median(dim=1).values.tolist()]
    net = ff.Net(layers, B, st.w_master, st.w_q, st.s_w, lookahead=look, theta_layer=theta)
    return {"what": "step", "st": st, "net": net, "ws": ws, "loss": loss, "good": good, "xp": xp, "xn": xn,
            "lam": case["lam"], "lr": LR[case["net"]], "step": 1}


def _run_step(s):
    ff.ff_train_step(s["net"], s["xp"], s["xn"], 2.0, s["lam"], s["lr"], SR_SEED, s["step"], s["loss"], s["good"], s["ws"])
    s["step"] += 1
    return {"loss": s["loss"], "goodness": s["good"], "w": s["st"].w_master, "wq": s["st"].w_q, "sw": s["st"].s_w}


# ---- one layer ---------------------------------------------------------------------------------------------------------

def _layer_state(case, layers, w):
    l, B = layers[0], case["batch"]
    d = ff.layer_desc(l, B)
    wq = torch.zeros((l.N, ff.ff_pitch(l.K)), dtype=torch.int8, device="cuda")
    sw = torch.zeros(1, device="cuda")
    ws = torch.empty(max(ff.WS_MIN_BYTES, ff.ff_layer_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
    ff.ff_quantize(w[0], l.N, l.K, ff.ROUND_NEAREST, 0, 0, wq, None, sw, ws)
    M = B * l.rows_per_sample
    rows, cols = (B, l.K) if l.kind == "dense" else (B * l.H * l.W, l.C_in)
    return {"what": case["what"], "lr": LR[case["net"]], "l": l, "d": d, "B": B, "M": M, "rows": rows, "cols": cols, "w": w[0], "wq": wq,
            "sw": sw, "ws": ws}


def _buffers(s):
    l, B, M = s["l"], s["B"], s["M"]
    i8 = lambda r, c: torch.zeros((r, ff.ff_pitch(c)), dtype=torch.int8, device="cuda")   # noqa: E731
    f = lambda *n: torch.zeros(n, device="cuda")                                          # noqa: E731
    return {"q": i8(s["rows"], s["cols"]), "q_t": i8(s["cols"], s["rows"]) if l.kind == "dense" else None, "s_a": f(1),
            "acc": torch.zeros((M, ff.ff_pitch32(l.N)), dtype=torch.int32, device="cuda"),
            "gsum": torch.zeros(B, dtype=torch.int64, device="cuda"), "vmax": torch.zeros(B, dtype=torch.int32, device="cuda"),
            "good": f(B), "coeff": f(B), "loss": f(1), "amax": f(1), "hq": i8(M, l.N),
            "hq_t": i8(l.N, M) if l.kind == "dense" else None, "s_h": f(1)}


def _forward(s, b, x, tag, sign, theta):
    ff.ff_quantize(x, s["rows"], s["cols"], ff.ROUND_STOCHASTIC, SR_SEED, tag, b["q"], b["q_t"], b["s_a"], s["ws"])
    ff.ff_layer_forward(s["d"], b["q"], s["wq"], b["acc"], b["gsum"], b["vmax"], s["ws"])
    ff.ff_goodness_loss(s["d"], b["gsum"], b["vmax"], b["s_a"], s["sw"], sign, theta, b["good"], b["coeff"], b["loss"],
                        b["amax"])


def _prepare_forward(case, layers, xp, xn, w):
    s = _layer_state(case, layers, w)
    b = _buffers(s)
    _forward(s, b, xp, 0, ff.PASS_POS, 2.0)
    s.update(b=b, x=xp, theta=_three_digits(b["good"].median().item()), step=1)
    return s


def _run_forward(s):
    b, l = s["b"], s["l"]
    _forward(s, b, s["x"], ff.ff_stream_tag(s["step"], 0, 0, ff.KIND_ACT), ff.PASS_POS, s["theta"])
    ff.ff_layer_handoff(s["d"], b["acc"], b["s_a"], s["sw"], b["good"], b["amax"], ff.ROUND_STOCHASTIC, SR_SEED,
                        ff.ff_stream_tag(s["step"], 1, 0, ff.KIND_ACT), b["hq"], b["hq_t"], b["s_h"])
    s["step"] += 1
    out = {n: b[n] for n in ("q", "s_a", "gsum", "vmax", "good", "coeff", "loss", "amax", "hq", "s_h")}
    out["acc"] = b["acc"][:, :l.N]
    if l.kind == "dense":
        out["q_t"], out["hq_t"] = b["q_t"], b["hq_t"]
    return out


def _prepare_backward(case, layers, xp, xn, w):
    s = _layer_state(case, layers, w)
    l, M = s["l"], s["M"]
    s["b"] = []
    theta = 2.0
    for i, (x, sign) in enumerate(((xp, ff.PASS_POS), (xn, ff.PASS_NEG))):
        b = _buffers(s)
        _forward(s, b, x, i, sign, theta)
        if i == 0:
            theta = _three_digits(b["good"].median().item())
            _forward(s, b, x, i, sign, theta)
        b["gy"] = torch.zeros((l.N, ff.ff_pitch(M)), dtype=torch.int8, device="cuda")
        b["s_g"] = torch.zeros(1, device="cuda")
        b["dw"] = torch.zeros((ff.ff_layer_dw_chunks(s["d"]), l.N, ff.ff_pitch32(l.K)), dtype=torch.int32, device="cuda")
        s["b"].append(b)
    s["step"] = 1
    return s


def _run_backward(s):
    l, d = s["l"], s["d"]
    for i, b in enumerate(s["b"]):
        ff.ff_layer_backward_local(d, b["acc"], b["vmax"], b["s_a"], s["sw"], b["coeff"], ff.ROUND_STOCHASTIC, SR_SEED,
                                   ff.ff_stream_tag(s["step"], 0, i, ff.KIND_GRAD), b["q_t"] if l.kind == "dense" else b["q"],
                                   b["gy"], b["s_g"], b["dw"], s["ws"])
    p, n = s["b"]
    ff.ff_layer_update(d, s["w"], p["dw"], p["s_g"], p["s_a"], n["dw"], n["s_g"], n["s_a"], s["lr"], 2 * s["B"], s["wq"],
                       s["sw"], s["ws"])
    s["step"] += 1
    return {"gy": [b["gy"] for b in s["b"]], "s_g": [b["s_g"] for b in s["b"]], "dw": [b["dw"][:, :, :l.K] for b in s["b"]],
            "w": s["w"], "wq": s["wq"], "sw": s["sw"]}


# ---- what a pass cannot do without -------------------------------------------------------------------------------------

def _macs(c):
    """Multiply-adds of one pass over one data set, forward only."""
    return sum(c["batch"] * l.rows_per_sample * l.N * l.K for l in _layers(c))


def work(case):
    layers, B = _layers(case), case["batch"]
    weights = sum(l.N * l.K for l in layers)
    x = B * layers[0].in_elems_per_sample
    y = B * layers[0].terms_per_sample
    if case["what"] == "forward":     # read x and int8 weights; write codes (dense: twice), accumulators, hand-off codes
        copies = 2 if layers[0].kind == "dense" else 1
        return {"bytes": 4 * x + weights + copies * x + 4 * y + copies * y, "flops": 2 * _macs(case)}
    if case["what"] == "backward":    # read accumulators and input codes; write gradient codes and accumulators; update
        return {"bytes": 2 * (4 * y + x + y + 4 * weights) + 9 * weights, "flops": 2 * 2 * _macs(case)}
    flops = 2 * 2 * 2 * _macs(case)   # both sets, forward and weight gradient
    if case.get("chain"):
        flops += 2 * 2 * sum(B * l.N * l.K for l in layers[1:])
    return {"bytes": 2 * 4 * x + 9 * weights + 4 * 2 * len(layers) * B, "flops": flops}


def tolerance(case):
    # Codes and integer accumulators are defined bit for bit (element-indexed rounding, integer sums): none may differ.
    # fp32 outputs are then short chains of single roundings, about 1e-6 together.  (Against 64 bits more is seen where a
    # code that falls the other way travels through later layers: 5e-5 in the goodness of a three-layer stack.)
    return {"rel": 4e-6, "max": 2e-5, "differ": 0.0}


# ---- the method in 64 bits ---------------------------------------------------------------------------------------------

def _key(tag):
    m = (1 << 64) - 1
    z = (SR_SEED + 0x9E3779B97F4A7C15 * (tag + 1)) & m
    z ^= z >> 30
    z = z * 0xBF58476D1CE4E5B9 & m
    z ^= z >> 27
    z = z * 0x94D049BB133111EB & m
    z ^= z >> 31
    return z & 0xFFFFFFFF


def _quantise(x, tag=None):
    """(codes as float64, scale) of a tensor; tag: stream of the stochastic rounding, None = to nearest even."""
    amax = float(x.abs().max())
    if amax < 2.0 ** -100:
        return torch.zeros_like(x), 1.0
    t = x * (127.0 / amax)
    if tag is None:
        return torch.round(t).clamp_(-127, 127), amax / 127.0
    v = torch.arange(x.numel(), device=x.device, dtype=torch.int64) ^ _key(tag)
    v ^= v >> 16
    v = v * 0x7FEB352D & 0xFFFFFFFF
    v ^= v >> 15
    v = v * 0x846CA68B & 0xFFFFFFFF
    v ^= v >> 16
    u = ((v >> 8).double() * 2.0 ** -24).reshape(x.shape)
    f = torch.floor(t)
    return (f + (u < t - f)).clamp_(-127, 127), amax / 127.0


def _tag(step, layer, p, kind):
    return step << 20 | layer << 4 | p << 2 | kind


def _patches(l, a, b0, b1):
    """Rows of the contraction for samples [b0, b1): [rows, K] (depthwise: [rows, C, taps])."""
    if l.kind == "dense":
        return a.reshape(-1, l.K)[b0:b1]
    a = a.reshape(-1, l.H, l.W, l.C_in)[b0:b1]
    a = torch.nn.functional.pad(a, (0, 0, l.pad, l.pad, l.pad, l.pad))
    ho, wo, s = l.H_out, l.W_out, l.stride
    taps = [a[:, i:i + (ho - 1) * s + 1:s, j:j + (wo - 1) * s + 1:s, :] for i in range(l.ksize) for j in range(l.ksize)]
    col = torch.stack(taps, dim=-1 if l.kind == "dwconv" else -2)
    return col.reshape(-1, l.C_in, l.K) if l.kind == "dwconv" else col.reshape(-1, l.K)


def _spans(l, B):
    per = max(1, int(2e8 // max(1, l.rows_per_sample * l.K * (l.C_in if l.kind == "dwconv" else 1))))
    return [(b, min(B, b + per)) for b in range(0, B, per)]


def _contract(l, a, wq, B):
    out = []
    for b0, b1 in _spans(l, B):
        col = _patches(l, a, b0, b1)
        out.append((col * wq).sum(-1) if l.kind == "dwconv" else col @ wq.t())
    return torch.cat(out)


def _weight_grad(l, a, g, B):
    dw, r = 0.0, l.rows_per_sample
    for b0, b1 in _spans(l, B):
        col, gg = _patches(l, a, b0, b1), g[b0 * r:b1 * r]
        dw = dw + ((col * gg.unsqueeze(-1)).sum(0) if l.kind == "dwconv" else gg.t() @ col)
    return dw


def _rows(v, l):
    return v.repeat_interleave(l.rows_per_sample).unsqueeze(1)


def _act(l, z):
    return z.clamp(min=0) if l.relu else z


def _loss(G, theta, p):
    x = (G - theta) * (1.0 if p else -1.0)
    return (1.0 if p else -1.0) * torch.sigmoid(x), torch.nn.functional.softplus(x).mean()


def _forward64(layers, wq, x, B, step, p):
    """Per layer: activities y, goodness G, int8 input codes and scale, the contraction in real units."""
    rec = []
    for i, l in enumerate(layers):
        src = i - 1 - l.input_back
        a, s_a = _quantise(x if src < 0 else rec[src]["out"], _tag(step, i, p, 0))
        r = {"a": a, "s_a": s_a, "z": _contract(l, a, wq[i][0], B) * (s_a * wq[i][1])}
        if l.role != "proj":
            z = r["z"]
            if l.skip == "identity":
                z = z + rec[i - 1]["a"].reshape(z.shape) * rec[i - 1]["s_a"]
            elif l.skip == "projection":
                z = z + rec[i - 2]["z"]
            r["y"] = _act(l, z)
            r["G"] = (r["y"] ** 2).reshape(B, -1).sum(1)
            n = _rows(r["G"].sqrt(), l)
            r["out"] = torch.where(n > 0, r["y"] / n, 0.0) if l.l2norm_out else r["y"]
        rec.append(r)
    return rec


def _step64(case, seed):
    layers, B, lam = _layers(case), case["batch"], case["lam"]
    xp, xn, w = _inputs(case, layers, seed)
    k, w = len(layers), [v.double() for v in w]
    wq = [_quantise(v) for v in w]
    xs = [xp.double(), xn.double()]
    rows = [[torch.zeros(B, device="cuda", dtype=torch.float64)] * 2 for _ in layers]
    start = [_forward64(layers, wq, xs[p], B, 0, p) for p in range(2)]
    # (the lower median, as torch takes it; layers without a goodness of their own keep 0)
    theta = [_three_digits(float(torch.cat([start[p][i].get("G", rows[i][0]) for p in range(2)]).float().median())) for i in range(k)]
    del start
    loss = torch.zeros((k, 2), device="cuda", dtype=torch.float64)
    good = torch.zeros((k, 2, B), device="cuda", dtype=torch.float64)
    grad = [0.0] * k
    for p in range(2):
        rec = _forward64(layers, wq, xs[p], B, 1, p)
        c = []
        for i, r in enumerate(rec):
            if "G" not in r:
                c.append(torch.zeros(B, device="cuda", dtype=torch.float64))
                continue
            ci, loss[i, p] = _loss(r["G"], theta[i], p)
            good[i, p] = r["G"]
            c.append(ci)
        S, E = 0.0, None
        for i in range(k - 1, -1, -1):
            l, r = layers[i], rec[i]
            if "G" not in r:
                continue
            if case.get("chain"):
                t = _rows(2 * c[i], l) * r["y"]
                live = (r["z"] > 0) if l.relu else torch.ones_like(r["z"], dtype=torch.bool)
                g = torch.where(live, t if E is None else t + lam * E, 0.0)
                h = torch.where(live, t if E is None else t + E, 0.0)
                if i:
                    hq, s_h = _quantise(h, _tag(1, i, p, 2))
                    E = hq @ wq[i][0] * (s_h * wq[i][1])
            else:
                g = _rows(2 * (c[i] + lam * S), l) * r["y"]
                S = S + c[i]
            gq, s_g = _quantise(g, _tag(1, i, p, 1))
            for t in [i] + ([i - 2] if l.skip == "projection" else []):
                grad[t] = grad[t] + _weight_grad(layers[t], rec[t]["a"], gq, B) * (s_g * rec[t]["s_a"])
    w = [v - LR[case["net"]] / (2 * B) * g.reshape(v.shape) for v, g in zip(w, grad)]
    return {"loss": loss, "goodness": good, "w": w, "wq": [None] * k,
            "sw": [torch.tensor([_quantise(v)[1]], dtype=torch.float64) for v in w]}


def exact(case, seed):
    if case["what"] == "step":
        return _step64(case, seed)
    layers, B = _layers(case), case["batch"]
    l = layers[0]
    xp, xn, w = _inputs(case, layers, seed)
    w0 = w[0].double()
    wq = [_quantise(w0)]
    one = lambda v: torch.tensor([float(v)], dtype=torch.float64)   # noqa: E731
    if case["what"] == "forward":
        theta = _three_digits(float(_contract_goodness(l, wq, xp, B, 0).float().median()))
        r = _forward64(layers, wq, xp.double(), B, 1, 0)[0]
        c, loss = _loss(r["G"], theta, 0)
        amax = r["out"].abs().max()
        out = {n: None for n in ("q", "gsum", "vmax", "hq", "acc")}
        if l.kind == "dense":
            out["q_t"] = out["hq_t"] = None
        out.update(s_a=one(r["s_a"]), good=r["G"], coeff=c, loss=one(loss), amax=one(amax), s_h=one(amax / 127.0))
        return out
    theta = _three_digits(float(_contract_goodness(l, wq, xp, B, 0).float().median()))
    grad, s_g = 0.0, []
    for p, x in enumerate((xp, xn)):
        a, s_a = _quantise(x.double(), p)
        y = _act(l, _contract(l, a, wq[0][0], B) * (s_a * wq[0][1]))
        c, _ = _loss((y ** 2).reshape(B, -1).sum(1), theta, p)
        gq, s = _quantise(_rows(2 * c, l) * y, _tag(1, 0, p, 1))
        grad = grad + _weight_grad(l, a, gq, B) * (s * s_a)
        s_g.append(one(s))
    v = w0 - LR[case["net"]] / (2 * B) * grad.reshape(w0.shape)
    return {"gy": [None] * 2, "s_g": s_g, "dw": [None] * 2, "w": v, "wq": None, "sw": one(_quantise(v)[1])}


def _contract_goodness(l, wq, x, B, tag):
    a, s_a = _quantise(x.double(), tag)
    return (_act(l, _contract(l, a, wq[0][0], B) * (s_a * wq[0][1])) ** 2).reshape(B, -1).sum(1)
