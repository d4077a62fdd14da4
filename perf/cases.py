"""The layers whose training (and inference) passes are timed, and how a program runs them.

A case is one convolution layer with the way it is driven:

  how = "step"    `LayerStep.run(overlap=None)`, the whole per-layer hot path of a training iteration: quantize a, W and
                  g_z, the clip search (search = True) or the clip value of an earlier search (search = False, the
                  Periodic Update of Sec.3.4), forward, backward-data and backward-weight convolution;
  how = "train"   the autograd modules (`Int8Conv2d`, `Int8Linear`): forward and backward pass of one layer;
  how = "eval"    the same modules without gradients: the forward pass of a network in use.

The shapes are layers of the networks of `paper_1912_12607_amd/inputs.py` (ResNet-18 / -50, MobileNetV2,
InceptionV3); values follow its recipe, drawn on the GPU.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1912_12607_amd.autograd import Int8Conv2d, Int8Linear
from paper_1912_12607_amd.inputs import Layer, default_ratios
from paper_1912_12607_amd.step import LayerStep

CANDIDATES = 32


def _case(name, how, N, C, H, K, R, S=None, stride=1, pad_h=None, pad_w=None, groups=1, search=True, first=False,
          x="relu", df=3.0, scale=1e-4, outliers=True, W=None):
    S = R if S is None else S
    c = dict(how=how, search=search, first=first, N=N, C=C, H=H, W=H if W is None else W, K=K, R=R, S=S, stride=stride,
             pad_h=R // 2 if pad_h is None else pad_h, pad_w=S // 2 if pad_w is None else pad_w, groups=groups,
             x=x, df=df, scale=scale, outliers=outliers)
    if name:
        c["name"] = name
    return c


def listed():
    mbv2 = dict(x="relu6", df=2.0, outliers=False)
    return [
        # the smallest step: a toy layer, nothing but launches and host time
        _case("tiny_3x3", "step", 2, 16, 16, 32, 3, x="normal", scale=1e-3),
        # the 3x3 layer of ResNet-18's first stage, clip searched in every iteration
        _case("r18_3x3_56", "step", 64, 64, 56, 64, 3),
        # a bottleneck's reducing 1x1 at 14 x 14, in an iteration that keeps its clip value
        _case("r50_1x1_reduce_14", "step", 128, 1024, 14, 256, 1, x="normal", scale=1e-3, search=False),
        # a bottleneck's 3x3 at 14 x 14: too few output tiles for large ones
        _case("r50_3x3_14", "step", 64, 256, 14, 256, 3),
        # the widest activations of ResNet-50 at the batch of a 288 GB device: 206 M gradient elements, streaming passes
        _case("r50_1x1_expand_56", "step", 256, 64, 56, 256, 1),
        # the first layer of a network: 3 channels, 7x7 under stride 2, no gradient of the images
        _case("r50_stem", "step", 64, 3, 224, 64, 7, stride=2, first=True),
        # MobileNetV2's depthwise 3x3, clip value kept
        _case("mbv2_depthwise_56", "step", 64, 144, 56, 144, 3, groups=144, search=False, **mbv2),
        # InceptionV3's 1x7 at 17 x 17 (odd image): the most arithmetic
        _case("inc_1x7_17", "step", 64, 768, 17, 768, 1, 7, x="normal", scale=1e-3),
        # InceptionV3's 5x5 branch at 35 x 35: odd image, 48 channels, even and odd remainders everywhere
        _case("inc_5x5_35", "step", 32, 48, 35, 64, 5, search=False),
        # a training pass through the module: the 3x3 that halves the image between two stages
        _case("train_3x3_s2_56", "train", 64, 128, 56, 128, 3, stride=2),
        # a classifier through the module: fully connected, with a bias
        _case("train_fc", "train", 256, 2048, 1, 1000, 1),
        # inference through the module: MobileNetV2's projecting 1x1, 24 output channels
        _case("eval_project_56", "eval", 64, 144, 56, 24, 1, **mbv2),
    ]


def _out(c):
    return (c["H"] + 2 * c["pad_h"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad_w"] - c["S"]) // c["stride"] + 1


def _sizes(c):
    P, Q = _out(c)
    nx = c["N"] * c["C"] * c["H"] * c["W"]
    nw = c["K"] * (c["C"] // c["groups"]) * c["R"] * c["S"]
    ny = c["N"] * c["K"] * P * Q
    return nx, nw, ny, ny * (nw // c["K"])


def _cost(c):
    w = work(c)
    return w["bytes"] / 4e12 + w["flops"] / 1e15


def draw(rng):
    """A layer of the listed kinds with sizes of its own: channels, image and total work spread over the logarithm of
    their ranges (the batch follows from them), odd sides and channel counts among them, no more work than the listed
    layers have."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def channels(lo, hi):
        v = log_int(lo, hi)
        return v if rng.random() < 0.3 else max(8, (v + 4) // 8 * 8)

    most = min(sorted(_cost(c) for c in listed())[-2], 5e-4)
    while True:
        how = rng.choice(["step", "step", "step", "step", "train", "eval"])
        kind = rng.choice(["1x1", "1x1", "3x3", "3x3", "depthwise", "line", "5x5", "stem", "fc"])
        target, H, W = math.exp(rng.uniform(math.log(1e-6), math.log(most))), log_int(5, 112), None
        if rng.random() < 0.25:
            W = max(5, H + rng.randint(-4, 4))
        C, K, stride, R, S, groups, first = channels(8, 1024), channels(8, 1024), 1, 1, 1, 1, False
        if kind == "3x3":
            R = S = 3
            stride = rng.choice([1, 1, 2])
        elif kind == "1x1":
            stride = rng.choice([1, 1, 1, 2])
        elif kind == "depthwise":
            R = S = 3
            groups = K = C
            stride = rng.choice([1, 1, 2])
        elif kind == "line":
            R, S = rng.choice([(1, 7), (7, 1), (1, 3), (3, 1)])
        elif kind == "5x5":
            R = S = 5
        elif kind == "stem":
            C, R = 3, rng.choice([3, 7])
            S, stride, first = R, 2, True
            K, H, W = channels(16, 96), log_int(32, 224), None
        elif kind == "fc":
            H = W = 1
            C, K = channels(64, 4096), channels(10, 4096)
        pad = 0 if (kind == "3x3" and rng.random() < 0.25) else None
        c = _case(None, how, 1, C, H, K, R, S, stride=stride, pad_h=pad, pad_w=pad, groups=groups, W=W,
                  search=how == "train" or rng.random() < 0.5, first=first and how == "step",
                  x=rng.choice(["relu", "relu6", "normal"]), df=rng.choice([2.0, 3.0]), scale=rng.choice([1e-4, 1e-3]),
                  outliers=rng.random() < 0.7)
        c["N"] = min(256, max(1, round(target / _cost(c))))
        if _cost(c) <= most:
            return c


def _inputs(c, seed):
    """x, w, g_z of the case: (clipped) normal activations, Kaiming-normal weights, heavy-tailed output gradients
    (Student-t with 2 or 3 degrees of freedom, 0.01 % of the entries a hundred times as large)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape):
        return torch.randn(shape, generator=gen, device="cuda")

    P, Q = _out(c)
    x = normal((c["N"], c["C"], c["H"], c["W"]))
    if c["x"] == "relu":
        x.clamp_(min=0.0)
    elif c["x"] == "relu6":
        x.clamp_(0.0, 6.0)
    cg = c["C"] // c["groups"]
    w = normal((c["K"], cg, c["R"], c["S"])) * math.sqrt(2.0 / (cg * c["R"] * c["S"]))
    g = None
    if c["how"] != "eval":
        shape = (c["N"], c["K"], P, Q)
        g = normal(shape)
        chi2 = normal(shape).square_()
        for _ in range(int(c["df"]) - 1):
            chi2.addcmul_(t := normal(shape), t)
        g.div_(chi2.div_(c["df"]).clamp_(min=1e-12).sqrt_()).mul_(c["scale"])
        if c["outliers"]:
            g.mul_(torch.where(torch.rand(shape, generator=gen, device="cuda") < 1e-4, 100.0, 1.0))
    return x, w, g


class _SameDraws:
    """Every backward pass with the same stochastic draws, so that passes can be compared with one another."""

    def next_seed(self):
        return 20


class _Conv(_SameDraws, Int8Conv2d):
    pass


class _Linear(_SameDraws, Int8Linear):
    pass


def prepare(case, seed):
    x, w, g = _inputs(case, seed)
    state = {"how": case["how"], "search": case["search"]}
    if case["how"] == "step":
        pad = (case["pad_h"], case["pad_w"])
        layer = Layer("layer", case["N"], case["C"], case["H"], case["W"], case["K"], case["R"], case["S"],
                      stride=(case["stride"], case["stride"]), pad=pad, groups=case["groups"])
        # the search's own d_c is what Eq.7 consumes: no second report from the quantizer
        st = LayerStep(layer, n_cand=CANDIDATES, requantize_deviation=False, input_grad=not case["first"])
        st.x.copy_(x)
        st.w.copy_(w)
        st.dy.copy_(g)
        st.ratios.copy_(torch.from_numpy(np.ascontiguousarray(default_ratios(CANDIDATES))))
        if not case["search"]:
            st.run(seed=1, search=True, overlap=None)      # the earlier iteration whose clip value is kept
        state["step"], state["dx"] = st, not case["first"]
        return state
    if case["H"] == 1 and case["W"] == 1 and case["R"] == 1 and case["S"] == 1 and case["groups"] == 1:
        layer = _Linear(case["C"], case["K"], bias=True, n_candidates=CANDIDATES)
        x, w = x.reshape(case["N"], case["C"]), w.reshape(case["K"], case["C"])
        g = None if g is None else g.reshape(case["N"], case["K"])
    else:
        layer = _Conv(case["C"], case["K"], (case["R"], case["S"]), stride=case["stride"], padding=(case["pad_h"], case["pad_w"]),
                      groups=case["groups"], bias=False, n_candidates=CANDIDATES)
    with torch.no_grad():
        layer.weight.copy_(w)
    state["layer"], state["g"] = layer, g
    state["x"] = x.requires_grad_(case["how"] == "train")
    return state


def run(state):
    if state["how"] == "step":
        st = state["step"]
        st.run(seed=7, search=state["search"], overlap=None)
        out = {"y": st.y, "dw": st.dw}
        if state["dx"]:
            out["dx"] = st.dx
        if state["search"]:
            out.update(clip=st.clip, d_c=st.dev_search, d_all=st.dev_all)
        return out
    layer = state["layer"]
    if state["how"] == "eval":
        with torch.no_grad():
            return layer(state["x"])
    y = layer(state["x"])
    params = list(layer.parameters())
    grads = torch.autograd.grad(y, [state["x"]] + params, state["g"])
    return {"y": y.detach(), "grads": grads, "d_c": layer.deviation}


def work(case):
    """Each fp32 tensor read or written once; two operations per multiply-accumulate and pass, and per gradient element
    and candidate of a clip search the scaling, the rounding and the two sums of Eq.6."""
    nx, nw, ny, macs = _sizes(case)
    if case["how"] == "eval":
        return {"bytes": 4 * (nx + nw + ny), "flops": 2 * macs}
    passes = 2 if case["first"] else 3
    nbytes = 4 * ((1 if case["first"] else 2) * nx + 2 * nw + 2 * ny)
    return {"bytes": nbytes, "flops": 2 * passes * macs + (6 * CANDIDATES * ny if case["search"] else 0)}


def tolerance(case):
    """Integer sums are exact on every path; an fp32 result is one of them scaled (Eq.2), two or three fp32 roundings:
    against the products in 64 bits 1.1e-7 at most over these layers (2-norm), 2.5e-8 where the scale happens to be exact."""
    return {"rel": 4e-7}
