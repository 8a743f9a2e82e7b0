"""The calls that users of the linear-attention layers make, as timed and compared cases.

A case is one pass through `torch_glue.Layer` (the Hedgehog map of Eq. 5) or `torch_glue.ReluLayer` (the weight-free map):
a forward call, or a training step (forward, then backward with the saved state).  Shapes are those of the converted
video models (Wan-1.3B at 480p, Wan-14B at 720p, CogVideoX-2B), of the small fp32 configuration, and of short clips and
tests; values follow the recipe of `synth.py`: activations N(0, 1)/sqrt(d) with a scale per head and tensor from
U(0.5, 2), optionally 0.1 % of the tokens at 20 times the magnitude, W~ ~ N(0, 1), upstream gradient ~ N(0, 0.1^2).
"""
import math

import torch

from paper_2510_08318_amd import torch_glue as G

RELU_EPS = 1e-6        # in the denominator of the ReLU map
OUTLIER_FRACTION = 0.001


def _case(name, *, map="hedgehog", mode="bf16", step="fwd", B=1, H=1, n=1, d=128, layout="bhnd", wgrads=False,
          blend=False, centred=False, outliers=False):
    """mode: bf16 (matrix-core arithmetic), f32 (fp32 tensors), f32math (bf16 tensors, fp32 arithmetic);
    step: fwd (one forward call) or train (forward and backward)."""
    case = dict(map=map, mode=mode, step=step, B=B, H=H, n=n, d=d, layout=layout, wgrads=wgrads, blend=blend,
                centred=centred, outliers=outliers)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # a short clip or a test input: a call whose time is launches and latency
        _case("fwd_small", H=4, n=1000, d=64),
        # inference, one layer of the 1.3B model at 832x480 (21 x 30 x 52 tokens)
        _case("fwd_wan1p3b_480p", H=12, n=32760),
        # inference, one layer of the 14B model at 1280x720 (21 x 45 x 80 tokens) with outlier tokens: the headline shape
        _case("fwd_wan14b_720p", H=40, n=75600, outliers=True),
        # inference, CogVideoX-2B (13 x 30 x 45 tokens, 30 heads of width 64), heads interleaved as the projections leave them
        _case("fwd_cogvideox", H=30, n=17550, d=64, layout="bnhd"),
        # post-training step of a converted layer, learnable feature maps
        _case("train_wan1p3b_480p", step="train", H=12, n=32760, wgrads=True),
        # a step of the selective-transfer stage: output mixed with the softmax branch, gradient of the mixing scalar
        _case("train_mixed_480p", step="train", H=12, n=32760, layout="bnhd", wgrads=True, blend=True),
        # a short ragged batch with frozen feature maps (no weight gradients)
        _case("train_short_ragged", step="train", B=2, H=6, n=4133, d=64),
        # the kernel-function ablation's ReLU map at the training shape
        _case("train_relu_480p", map="relu", step="train", H=12, n=32760),
        # inputs whose map is nearly uniform need the centred operands; a quarter of the 480p clip
        _case("train_centred", step="train", H=12, n=8190, wgrads=True, centred=True),
        # the fp32 configuration: a small reference step
        _case("f32_train_small", mode="f32", step="train", H=2, n=1024, d=64, wgrads=True),
        # fp32 tensors at the 1.3B shape, inference
        _case("f32_fwd_480p", mode="f32", H=12, n=32760),
        # bf16 tensors with fp32 arithmetic, the mode for numerically delicate phases, at the training shape
        _case("f32math_train_480p", mode="f32math", step="train", H=12, n=32760, wgrads=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    mode = rng.choices(("bf16", "f32", "f32math"), (0.7, 0.12, 0.18))[0]
    step = rng.choice(("fwd", "train"))
    relu = rng.random() < 0.2
    d = rng.choice((64, 128))
    # head-token limits that keep a drawn case below the largest listed one of its kind
    most = 120_000 if mode != "bf16" else 3_000_000 if step == "fwd" else 390_000
    head_tokens = _log_int(rng, 500, most * 128 // d if mode != "bf16" or step == "train" else most)
    B = rng.choice((1, 1, 1, 2))
    H = min(_log_int(rng, 1, 40), max(1, head_tokens // B))
    n = max(32, min(75600, head_tokens // (B * H)))
    hedgehog = not relu
    return _case(None, map="relu" if relu else "hedgehog", mode=mode, step=step, B=B, H=H, n=n, d=d,
                 layout=rng.choice(("bhnd", "bnhd")), wgrads=hedgehog and step == "train" and rng.random() < 0.6,
                 blend=hedgehog and rng.random() < 0.2, centred=hedgehog and mode == "bf16" and rng.random() < 0.15)


def _dtype(case):
    return torch.float32 if case["mode"] == "f32" else torch.bfloat16


def _inputs(case, seed):
    """The stored tensors, on the GPU, in the case's layout."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    dt = _dtype(case)
    rows = None
    if case["outliers"]:
        count = int(math.ceil(OUTLIER_FRACTION * n))
        rows = torch.randperm(n, generator=gen, device="cuda")[:count]

    def tokens(std, scaled):
        x = torch.empty((B, H, n, d), dtype=dt, device="cuda")
        scale = torch.rand((B, H), generator=gen, device="cuda") * 1.5 + 0.5 if scaled else torch.ones((B, H), device="cuda")
        for b in range(B):
            for h in range(H):
                t = torch.randn((n, d), generator=gen, device="cuda") * (std * scale[b, h])
                if scaled and rows is not None:
                    t[rows] *= 20.0
                x[b, h] = t.to(dt)
        return x.permute(0, 2, 1, 3).contiguous() if case["layout"] == "bnhd" else x

    x = {name: tokens(1.0 / math.sqrt(d), True) for name in ("q", "k", "v")}
    if case["map"] == "hedgehog":
        for name in ("wq", "wk"):
            x[name] = torch.randn((H, d, d // 2), generator=gen, device="cuda").to(dt)
    if case["step"] == "train":
        x["dout"] = tokens(0.1, False)
    if case["blend"]:
        x["s"] = tokens(0.1, False)                                # the softmax branch's output
        x["r"] = torch.rand(1, generator=gen, device="cuda") * 0.8 + 0.1
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    f32_math = case["mode"] == "f32math"
    if case["map"] == "relu":
        layer = G.ReluLayer(case["H"], case["d"], case["B"], case["n"], _dtype(case), layout=case["layout"], f32_math=f32_math)
    else:
        layer = G.Layer(x["wq"], x["wk"], case["B"], case["n"], want_wgrads=case["wgrads"], layout=case["layout"],
                        f32_math=f32_math, centred=case["centred"])
    dr = None
    if case["blend"]:
        dr = torch.zeros(1, device="cuda") if case["step"] == "train" else None
        layer.set_blend(x["s"], x["r"], dr)
    return {"train": case["step"] == "train", "layer": layer, "x": x, "dr": dr}


def run(state):
    layer, x = state["layer"], state["x"]
    res = {"out": layer.forward(x["q"], x["k"], x["v"]), "state": layer.state}
    if state["train"]:
        res["dq"], res["dk"], res["dv"] = layer.backward(x["q"], x["k"], x["v"], x["dout"])
        if getattr(layer, "dwq", None) is not None:
            res["dwq"], res["dwk"] = layer.dwq, layer.dwk
        if state["dr"] is not None:
            res["dr"] = state["dr"]
    return res


def work(case):
    """Bytes: each tensor of a call read or written once (forward: q, k, v, out; backward: q, k, v, dout, dq, dk, dv; the
    softmax branch once per call); flops: the contractions of Eq. 3 and Eq. 5 and of their derivatives."""
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    head_tokens, train, relu = B * H * n, case["step"] == "train", case["map"] == "relu"
    esz = 4 if case["mode"] == "f32" else 2
    tensors = 4 + (7 if train else 0) + ((2 if train else 1) if case["blend"] else 0)
    weights = 0 if relu else 2 * H * d * (d // 2) * (esz + (4 if case["wgrads"] else 0))
    flops = (4 if relu else 6) * d * d                               # (projections,) phi(k)^T v, phi(q) S
    if train:
        flops += (8 if relu else 12 + (2 if case["wgrads"] else 0)) * d * d
    return {"bytes": tensors * head_tokens * d * esz + B * H * (d + 1) * d * 4 + weights, "flops": flops * head_tokens}


def tolerance(case):
    # About four times the distance of the outputs from exact().  fp32 tensors: 1.2e-6 (2-norm) and 1.6e-5 (largest) for the
    # weight gradients, the longest sums.  bf16 tensors: 1.7e-3 and 1e-2, the bf16 store of the results.
    return {"rel": 5e-6, "max": 6e-5} if case["mode"] == "f32" else {"rel": 7e-3, "max": 4e-2}


def _phi(x, w, relu):
    if relu:
        return torch.relu(x)
    u = x @ w
    return torch.cat((torch.softmax(u, -1), torch.softmax(-u, -1)), -1)


def exact(case, seed):
    x = _inputs(case, seed)
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    relu, train, blend = case["map"] == "relu", case["step"] == "train", case["blend"]
    bnhd = case["layout"] == "bnhd"

    def head(t, b, h):
        return (t[b, :, h] if bnhd else t[b, h]).double()

    def like(t):
        return torch.empty(t.shape, dtype=torch.float64, device="cuda")

    res = {"out": like(x["q"]), "state": torch.empty((B, H, d + 1, d), dtype=torch.float64, device="cuda")}
    if train:
        res.update({g: like(x["q"]) for g in ("dq", "dk", "dv")})
        if case["wgrads"]:
            res.update({g: torch.zeros((H, d, d // 2), dtype=torch.float64, device="cuda") for g in ("dwq", "dwk")})
        if blend:
            # a single number: its distance from 64 bits is one draw of the rounding noise (2e-7 to 5e-5 over the ranges),
            # which says nothing about precision; tolerance() holds it to the result itself
            res["dr"] = None
    r = x["r"].double().clamp(0, 1) if blend else None
    for b in range(B):
        for h in range(H):
            q, k, v = [head(x[t], b, h).requires_grad_(train) for t in ("q", "k", "v")]
            wq, wk = [None if relu else x[t][h].double().requires_grad_(train) for t in ("wq", "wk")]
            fk, fq = _phi(k, wk, relu), _phi(q, wq, relu)
            S, z = fk.t() @ v, fk.sum(0)
            o = (fq @ S) / ((fq @ z) + (RELU_EPS if relu else 0.0))[:, None]
            if blend:
                o = r * head(x["s"], b, h) + (1 - r) * o
            (res["out"][b, :, h] if bnhd else res["out"][b, h]).copy_(o.detach())
            res["state"][b, h, :d], res["state"][b, h, d] = S.detach(), z.detach()
            if train:
                wanted = [q, k, v] + ([] if relu else [wq, wk])
                grads = list(torch.autograd.grad(o, wanted, head(x["dout"], b, h)))
                for name in ("dq", "dk", "dv"):
                    (res[name][b, :, h] if bnhd else res[name][b, h]).copy_(grads.pop(0))
                if not relu:
                    gq, gk = grads.pop(0), grads.pop(0)
                    if case["wgrads"]:
                        res["dwq"][h] += gq
                        res["dwk"][h] += gk
    return res
