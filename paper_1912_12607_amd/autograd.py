"""PyTorch autograd plug-in over the C ABI: INT8 convolution and fully connected layers whose forward,
backward-data and backward-weight passes run on int8 codes (Sec.3.1 Eq.1-3, Sec.3.4), with the
gradient clip chosen by the Direction Sensitive Gradient Clipping search, the layer's deviation d_c
exposed for Deviation Counteractive LR Scaling (Sec.3.5 Eq.7), and `replace_modules()`, the
"automatic match and replacement" of a model's convolution and fully connected layers by their 8-bit
counterparts (Sec.3.6 item 1).

Plumbing only: every arithmetic step of the INT8 path is one of the library's entry points; torch
supplies device memory, the stream and the autograd graph (and adds the fp32 bias, which like the
normalisation layers stays unquantized, Sec.4).  CUDA(ROCm) tensors, fp32, contiguous NCHW.
"""
from __future__ import annotations

import zlib

import numpy as np
import torch

from . import binding as B
from .inputs import default_ratios


class _LayerBuffers:
    """Device buffers of one layer at one input shape, allocated once and kept: scratch, the codes of
    the weights and of the output gradient, the scalars.  The codes of the activations are the one
    thing a forward pass must keep until its backward pass: they come from a small pool per shape
    (taken in forward, handed back in backward), so a layer called several times before its backward
    passes keeps each call's codes apart, and a steady training loop allocates nothing."""

    def __init__(self, layer, x_shape, dev):
        N, C, H, W = x_shape
        K, Cg, R, S = layer.weight_shape
        if C != Cg * layer.groups:      # (the library takes the filters' channel count from the descriptor)
            raise RuntimeError(f"input of {C} channels in a layer of {Cg * layer.groups}")
        self.desc = B.make_desc(N, C, H, W, K, R, S, layer.stride, layer.padding, layer.groups)
        depthwise = layer.groups != 1
        self.act_kind = B.ACT_PLANAR if depthwise else B.ACT
        self.wgt_kind = B.WGT_PLANAR if depthwise else B.WGT
        P = (H + 2 * layer.padding[0] - R) // layer.stride[0] + 1
        Q = (W + 2 * layer.padding[1] - S) // layer.stride[1] + 1
        self.x_shape, self.w_shape, self.y_shape = (N, C, H, W), (K, Cg, R, S), (N, K, P, Q)
        i8, f32, u8 = torch.int8, torch.float32, torch.uint8
        self.dev = dev
        self.wq = torch.empty(B.int8t_code_bytes(self.w_shape, self.wgt_kind), dtype=i8, device=dev)
        self.dyq = torch.empty(B.int8t_code_bytes(self.y_shape, self.act_kind), dtype=i8, device=dev)
        self.sw = torch.empty(1, dtype=f32, device=dev)
        self.sdy = torch.empty(1, dtype=f32, device=dev)
        self.xq_bytes = B.int8t_code_bytes(self.x_shape, self.act_kind)
        self.xq_pool = []
        n_y = N * K * P * Q
        nq = B.int8t_quantize_batch_workspace_bytes(
            [(None, self.x_shape, self.act_kind, None, None, None), (None, self.w_shape, self.wgt_kind, None, None, None)])
        nbytes = max(256, nq, B.int8t_workspace_bytes(B.OP_CONV_FWD, self.desc),
                     B.int8t_workspace_bytes(B.OP_DSGC, None, n_y, layer.ratios.numel()),
                     B.int8t_quantize_workspace_bytes(self.y_shape, self.act_kind),
                     B.int8t_workspace_bytes(B.OP_CONV_BWD_WEIGHT, self.desc),
                     B.int8t_workspace_bytes(B.OP_CONV_BWD_DATA, self.desc))
        self.ws = torch.empty(nbytes, dtype=u8, device=dev)
        # (one scratch for all calls: they follow each other on one stream, and passes that share a launch use one scratch at most)
        self._fwd = B.layer_buffers(wq=self.wq, sw=self.sw, ws_quant=self.ws, ws_fwd=self.ws)
        self._bwd = B.layer_buffers(wq=self.wq, dyq=self.dyq, sw=self.sw, sdy=self.sdy, ws_dy=self.ws, ws_bwd_data=self.ws,
                                    ws_bwd_weight=self.ws)
        self.w_numel = K * Cg * R * S
        # Sums over the rows of g_z in the call of the backward passes.  64 columns are one block there, whatever the rows: us with
        # the sums inside / behind it (torch.sum), search included, 1000 columns: 256 rows 33.6, 41.8; 1024: 45.4, 52.3; 2048: 58.7,
        # 60.1; 4096: 91.8, 85.7; 65535: 1131, 615; 64 columns: 1024 rows 31.4, 36.6; 2048: 38.3, 39.2; 8192: 94.9, 52.8.
        # (without the search 1000 columns: 1024 rows 32.5, 34.1; 2048: 43.4, 41.2)
        self.sums = P * Q == 1 and N <= 1024

    def take_xq(self):
        if self.xq_pool:
            return self.xq_pool.pop()
        return (torch.empty(self.xq_bytes, dtype=torch.int8, device=self.dev),
                torch.empty(1, dtype=torch.float32, device=self.dev))

    def give_xq(self, pair):
        self.xq_pool.append(pair)


def _device(t):
    """Address of a tensor for the library."""
    assert t.is_cuda and t.is_contiguous(), "device-resident contiguous tensors only"
    return t.data_ptr()


class _Int8ConvFn(torch.autograd.Function):
    """One layer's forward and backward pass.  x in the module's own shape (N,C,H,W, or (.., C) where the layer is fully
    connected: `linear`), w in the parameter's; a bias that is given is added here, and its gradient is formed with the others, so
    that the layer is one node of the graph and each direction one call of the library.  (As a chain of nodes -- two reshapes, a
    view of the weights, the addition -- with the library called once per kernel group, a pass of a 2048 -> 1000 classifier at batch
    256 kept the host busy for 224 us, 75 forward and 142 backward, where the GPU needs 75; now 36 and 62.)"""

    @staticmethod
    def forward(ctx, x, w, layer, keep, bias, linear):
        x = x.contiguous()
        w = w.contiguous()
        x_shape = tuple(x.shape)
        buf = layer.buffers((x.numel() // layer.in_channels, layer.in_channels, 1, 1) if linear else x_shape, x.device)
        if w.numel() != buf.w_numel:
            raise RuntimeError(f"weight of {w.numel()} elements in a layer of {buf.w_numel}")
        xq, sx = buf.take_xq()
        y = torch.empty(x_shape[:-1] + (buf.y_shape[1],) if linear else buf.y_shape, dtype=torch.float32, device=x.device)
        # codes of the activations and the weights (one absmax launch, one quantize launch) and the convolution; where no backward
        # pass will come for the codes, the library may do without them
        b = B.LayerBuffers.from_buffer_copy(buf._fwd)
        b.x, b.w, b.xq, b.sx, b.y = _device(x), _device(w), xq.data_ptr(), sx.data_ptr(), y.data_ptr()
        if keep:
            B.int8t_layer_step(buf.desc, b, B.STEP_ABSMAX | B.STEP_QUANT_XW | B.STEP_FWD)
        else:
            B.int8t_layer_infer(buf.desc, b)
        if bias is not None:
            y.add_(bias if linear else bias.view(1, -1, 1, 1))
        if keep:      # a backward pass will come for the codes
            ctx.layer, ctx.buf, ctx.xq = layer, buf, (xq, sx)
            ctx.w_version = layer.weight._version
            ctx.x_shape, ctx.w_shape = x_shape, tuple(w.shape)
        else:
            buf.give_xq((xq, sx))
        ctx.linear = linear
        return y

    @staticmethod
    def backward(ctx, dy):
        dy = dy.contiguous()
        want_x, want_w, want_b = ctx.needs_input_grad[0], ctx.needs_input_grad[1], ctx.needs_input_grad[4]
        batch_dims = tuple(range(dy.dim() - 1)) if ctx.linear else (0, 2, 3)
        if not (want_x or want_w):           # a frozen layer with a trained bias
            return None, None, None, None, dy.sum(batch_dims) if batch_dims else dy, None
        layer, buf = ctx.layer, ctx.buf
        xq, sx = ctx.xq
        n_y = dy.numel()
        seed = layer.next_seed()
        if layer.clip is None:
            layer.clip = torch.empty(1, dtype=torch.float32, device=dy.device)
            layer.deviation = torch.zeros(1, dtype=torch.float64, device=dy.device)
        parts = B.STEP_QUANT_G
        step = B.LayerBuffers.from_buffer_copy(buf._bwd)
        step.dy, step.xq, step.sx = _device(dy), xq.data_ptr(), sx.data_ptr()
        step.clip = _device(layer.clip)
        # Periodic Update (Sec.3.4): the clip value is searched every `dsgc_period` backward passes
        if layer.backward_calls % layer.dsgc_period == 0:
            J = layer.ratios.numel()
            refine = layer.dsgc_refine
            if refine:
                B.int8t_dsgc_clip(dy, n_y, layer.ratios, J, B.ROUND_STOCHASTIC, seed, layer.clip, layer.deviation, layer.dev_all, buf.ws)
            else:
                parts |= B.STEP_PREPARE | B.STEP_SEARCH       # with the passes, below
                step.ratios, step.n_cand = _device(layer.ratios), J
                step.dev_search = _device(layer.deviation)
            # Refinement of the clip value (Sec.3.4 learns c by descending d_c; no step size is given): further
            # sweeps over J candidates spaced geometrically around the last winner, the window shrinking by the
            # factor J / 2 each time.  The winner itself is candidate J / 2, so d_c never rises.  The ratios are
            # formed on the device (no host round trip): winner's ratio times 2^((j - J/2) * w / J), capped at 1.
            ratios, width = layer.ratios, layer.ratio_step
            for _ in range(refine):
                best = torch.argmin(layer.dev_all[:J])
                ratios = torch.clamp(ratios[best] * layer.refine_factors(width), max=1.0)
                B.int8t_dsgc_clip(dy, n_y, ratios, J, B.ROUND_STOCHASTIC, seed,
                                  layer.clip, layer.deviation, layer.dev_all, buf.ws)
                width = 2.0 * width / J
            layer.last_ratios = ratios          # the candidates of the last sweep (the grid itself without refinement)
        else:
            step.dev_final = _device(layer.deviation)          # Eq.6 of the codes actually produced with the kept clip
        layer.backward_calls += 1
        if layer.weight._version != ctx.w_version:
            # the weights changed between this layer's forward and backward pass (an optimizer step in
            # between): the codes of W the forward used are gone, quantize the current ones again
            B.int8t_quantize(layer.weight.detach().contiguous().view(buf.w_shape), buf.w_shape, buf.wgt_kind, None, B.ROUND_NEAREST_EVEN, 0,
                             buf.wq, buf.sw, None, buf.ws)
        # the bias gradient: sums over the rows in the same call, where nobody wants to differentiate them again and a block can walk
        # the rows of its columns (_LayerBuffers.sums)
        db = sums = None
        if want_b and buf.sums and not torch.is_grad_enabled():
            db = sums = torch.empty(buf.y_shape[1], dtype=torch.float32, device=dy.device)
        elif want_b:
            db = dy.sum(batch_dims) if batch_dims else dy
        # the search, codes of g_z and the passes wanted, in one call (it lets passes that do not fill the chip share a launch)
        dx = dw = None
        if want_x:
            dx = torch.empty(ctx.x_shape, dtype=torch.float32, device=dy.device)
            step.dx = dx.data_ptr()
            parts |= B.STEP_BWD_DATA
        if want_w:
            dw = torch.empty(ctx.w_shape, dtype=torch.float32, device=dy.device)
            step.dw = dw.data_ptr()
            parts |= B.STEP_BWD_WEIGHT
        B.int8t_layer_backward(buf.desc, step, parts, seed, sums)
        buf.give_xq((xq, sx))
        ctx.xq = None
        return dx, dw, None, None, db, None


_functorch_active = getattr(torch._C, "_are_functorch_transforms_active", lambda: False)


def _plain_eager() -> bool:
    """No transformation looks at the single operations of the layer: no functorch level, forward-mode level or tracer."""
    return (getattr(torch.autograd.forward_ad, "_current_level", -1) < 0 and not _functorch_active()
            and not torch.jit.is_tracing() and not torch.compiler.is_compiling())


def _pair(v):
    return (v, v) if isinstance(v, int) else tuple(v)


class Int8Conv2d(torch.nn.Module):
    """Drop-in for `torch.nn.Conv2d` (groups 1 or depthwise, dilation 1, zero padding).  The bias, if
    any, stays fp32 and is added to the dequantized result.  After a backward pass `deviation` holds
    d_c of this layer's output gradient (device, fp64) and `dclr_scale()` the factor phi(d_c) of Eq.7
    to multiply this layer's learning rate with."""

    def __init__(self, in_channels, out_channels, kernel_size, stride=1, padding=0, groups=1, bias=False,
                 n_candidates: int = 32, dsgc_period: int = 1, dsgc_refine: int = 0, seed: int | None = None,
                 device="cuda:0", name: str = ""):
        """dsgc_refine: sweeps that refine the clip value around the winner of the candidate grid (0: the grid only)."""
        super().__init__()
        self.in_channels, self.out_channels = in_channels, out_channels
        self.kernel_size, self.stride, self.padding, self.groups = _pair(kernel_size), _pair(stride), _pair(padding), groups
        assert groups == 1 or (groups == in_channels == out_channels), "groups 1 or depthwise"
        fan_in = (in_channels // groups) * self.kernel_size[0] * self.kernel_size[1]
        w = torch.randn(out_channels, in_channels // groups, *self.kernel_size, device=device) * (2.0 / fan_in) ** 0.5
        self.weight = torch.nn.Parameter(w)
        self.weight_shape = tuple(w.shape)      # K, C/groups, R, S (the Parameter of Int8Linear is K, C)
        self.bias = torch.nn.Parameter(torch.zeros(out_channels, device=device)) if bias else None
        self.ratios = torch.from_numpy(np.ascontiguousarray(default_ratios(n_candidates))).to(device)
        self.dsgc_period = max(1, int(dsgc_period))
        self.dsgc_refine = max(0, int(dsgc_refine))
        # log2 of the spacing of the grid's neighbours around a winner: the first refinement spans one grid step each way
        r = default_ratios(n_candidates)
        self.ratio_step = 2.0 * float(np.log2(r[0] / r[1])) if n_candidates > 1 else 1.0
        self.dev_all = torch.zeros(B.MAX_CANDIDATES, dtype=torch.float64, device=device) if self.dsgc_refine else None
        self._j = torch.arange(n_candidates, dtype=torch.float32, device=device) - float(n_candidates // 2)
        self.backward_calls = 0
        self.last_ratios = None
        self.clip = None
        self.deviation = None
        # Stream of seeds of the stochastic rounding (Eq.3): starts at a hash of the layer's name, so that
        # the layers of a model do not share their draws, and advances by one per backward pass.
        self._seed = int(seed) if seed is not None else (zlib.crc32(name.encode()) << 20 if name else 0)
        self._buffers = {}

    def buffers(self, x_shape, dev) -> _LayerBuffers:
        key = (x_shape, str(dev))
        if key not in self._buffers:
            self._buffers[key] = _LayerBuffers(self, x_shape, dev)
        return self._buffers[key]

    def refine_factors(self, width: float) -> torch.Tensor:
        """2^((j - J/2) * width / J), j = 0..J-1, fp32 on the layer's device (factor 1 at j = J/2)."""
        return torch.exp2(self._j * (width / self._j.numel()))

    def next_seed(self) -> int:
        self._seed += 1
        return self._seed

    def forward(self, x):
        return self._run(x, False)

    def _run(self, x, linear):
        w, bias = self.weight, self.bias
        keep = torch.is_grad_enabled() and (x.requires_grad or w.requires_grad)
        if (_plain_eager() and (x.dim() >= 1 and x.shape[-1] == self.in_channels if linear else x.dim() == 4)
                and (bias is None or (bias.dim() == 1 and bias.shape[0] == self.out_channels and bias.is_cuda and bias.dtype is torch.float32))):
            return _Int8ConvFn.apply(x, w, self, keep, bias, linear)
        # the same as single operations
        lead = x.shape[:-1]
        y = _Int8ConvFn.apply(x.reshape(-1, self.in_channels, 1, 1) if linear else x, w.view(self.weight_shape), self, keep, None, False)
        if bias is not None:
            y = y + bias.view(1, -1, 1, 1)
        return y.reshape(*lead, self.out_channels) if linear else y

    def dclr_scale(self, alpha: float = 20.0, beta: float = 0.1) -> float:
        """phi(d_c) = max(exp(-alpha d_c), beta) for the last backward pass (reads d_c back)."""
        if self.deviation is None:
            return 1.0
        return B.int8t_dclr_scale(float(self.deviation.item()), alpha, beta)


class Int8Linear(Int8Conv2d):
    """Drop-in for `torch.nn.Linear`: the 8-bit fully connected layer of Sec.3.6 item 1, run as the
    1 x 1 convolution of a 1 x 1 image through the same entry points.  Input (..., in_features)."""

    def __init__(self, in_features, out_features, bias=True, **kw):
        super().__init__(in_features, out_features, 1, bias=bias, **kw)
        self.in_features, self.out_features = in_features, out_features
        self.weight = torch.nn.Parameter(self.weight.data.view(out_features, in_features))    # nn.Linear's shape

    def forward(self, x):
        return self._run(x, True)


def replace_modules(model: torch.nn.Module, n_candidates: int = 32, dsgc_period: int = 1, skip=(), dsgc_refine: int = 0) -> int:
    """Swaps, in place, every `nn.Conv2d` the library covers (groups 1 or depthwise, dilation 1, zero
    padding) and every `nn.Linear` of `model` for its INT8 counterpart, keeping the parameters (the
    very Parameter objects, so optimizers and state dicts keep working) -- the automatic match and
    replacement of Sec.3.6 item 1.  Modules whose qualified name is in `skip`, and convolutions the
    library does not cover (other group counts, dilation, non-zero padding modes), are left alone.
    Returns the number of modules replaced."""
    count = 0
    for qual, parent in list(model.named_modules()):
        for child_name, m in list(parent.named_children()):
            full = f"{qual}.{child_name}" if qual else child_name
            if full in skip or isinstance(m, Int8Conv2d):
                continue
            new = None
            if isinstance(m, torch.nn.Conv2d):
                ok = (m.dilation == (1, 1) and m.padding_mode == "zeros" and not isinstance(m.padding, str)
                      and (m.groups == 1 or m.groups == m.in_channels == m.out_channels))
                if ok:
                    new = Int8Conv2d(m.in_channels, m.out_channels, m.kernel_size, m.stride, m.padding, m.groups,
                                     bias=False, n_candidates=n_candidates, dsgc_period=dsgc_period, dsgc_refine=dsgc_refine,
                                     device=m.weight.device, name=full)
            elif isinstance(m, torch.nn.Linear):
                new = Int8Linear(m.in_features, m.out_features, bias=False, n_candidates=n_candidates,
                                 dsgc_period=dsgc_period, dsgc_refine=dsgc_refine, device=m.weight.device, name=full)
            if new is None:
                continue
            new.weight = m.weight
            new.bias = m.bias
            new.train(m.training)
            setattr(parent, child_name, new)
            count += 1
    return count


class DclrSGD(torch.optim.SGD):
    """SGD whose learning rate is scaled per INT8 layer by phi(d_c) of that layer's last backward
    pass: Deviation Counteractive LR Scaling, Sec.3.5 Eq.7.  Parameters that belong to no INT8 layer
    (and the fp32 biases) keep the base rate.  `step()` reads all layers' d_c back in ONE copy."""

    def __init__(self, model: torch.nn.Module, lr: float, alpha: float = 20.0, beta: float = 0.1, **sgd_kwargs):
        self.alpha, self.beta = alpha, beta
        self._layers = [m for m in model.modules() if isinstance(m, Int8Conv2d)]
        int8_ids = {id(m.weight) for m in self._layers}
        rest = [p for p in model.parameters() if id(p) not in int8_ids]
        groups = [{"params": [m.weight], "base_lr": lr} for m in self._layers]
        if rest:
            groups.append({"params": rest, "base_lr": lr})
        super().__init__(groups, lr=lr, **sgd_kwargs)

    def set_lr(self, lr: float):
        """New base rate (schedulers act on this, the DCLR factor is applied on top)."""
        for g in self.param_groups:
            g["base_lr"] = lr

    def deviations(self):
        """d_c of every INT8 layer's last backward pass (0 where none has run), one device-to-host copy."""
        have = [m.deviation for m in self._layers if m.deviation is not None]
        vals = iter(torch.cat(have).cpu().tolist()) if have else iter(())
        return [next(vals) if m.deviation is not None else 0.0 for m in self._layers]

    @torch.no_grad()
    def step(self, closure=None):
        for g, d in zip(self.param_groups, self.deviations()):
            g["lr"] = g["base_lr"] * B.int8t_dclr_scale(d, self.alpha, self.beta)
        for g in self.param_groups[len(self._layers):]:
            g["lr"] = g["base_lr"]
        return super().step(closure)
