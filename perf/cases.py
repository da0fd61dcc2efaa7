"""The work that programs have this library do, as cases to be timed and compared.

Every case is one training step of a part of a network through the public
entry points: F for each micro-batch, then F' (where checkpointed), B and the
gradient accumulation, as a stage of a pipeline runs it (kinds "layer",
"unet-stage", "cells"), or a whole tgp_pipeline_step with its loss (kinds
"stack" and "unet").  Inputs are made on the GPU from the seed: activations of
hidden layers are rectified normals, images, targets and upstream gradients
normals, weights He-normal, biases 0.1 of a normal.
"""
import math

import torch

import paper_2004_09910_amd as tgp

CONV3, CONV1, DW3 = 0, 1, 2                    # tgp_kind
NOPRO, POOL, UPCAT = 0, 1, 2                   # tgp_prologue
MODES = {"always": tgp.CKPT_ALWAYS, "except_last": tgp.CKPT_EXCEPT_LAST, "never": tgp.CKPT_NEVER}
DT = {"bf16": (tgp.BF16, torch.bfloat16), "fp32": (tgp.FP32, torch.float32)}


# ---------------------------------------------------------------- the cases

def _layer(name, kind, cin, cout, h, w, b, m, group, mode="never", dtype="bf16", pool=False,
           relu=True, bias=True):
    """One layer as a stage: `b` samples a micro-batch, `m` micro-batches,
    `group` of them a call; h x w is the size of the convolution (a pooled
    layer's input is twice that)."""
    c = {"kind": "layer", "op": kind, "cin": cin, "cout": cout, "h": h, "w": w, "b": b, "m": m,
         "group": group, "mode": mode, "dtype": dtype, "pool": pool, "relu": relu, "bias": bias}
    return dict(c, name=name) if name else c


def _cells(name, cells, c, h, w, b, m, group, mode):
    c = {"kind": "cells", "cells": cells, "c": c, "h": h, "w": w, "b": b, "m": m, "group": group,
         "mode": mode, "dtype": "bf16"}
    return dict(c, name=name) if name else c


def _unet_stage(name, base, hw, layers, b, m, group, mode):
    """The first `layers` layers of a 5-level U-Net's encoder."""
    c = {"kind": "unet-stage", "base": base, "hw": hw, "layers": layers, "b": b, "m": m,
         "group": group, "mode": mode, "dtype": "bf16"}
    return dict(c, name=name) if name else c


def _step(name, kind, dtype, mode, b, m, n, lanes, **net):
    c = dict(net, kind=kind, dtype=dtype, mode=mode, b=b, m=m, n=n, lanes=lanes)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest step there is a configuration of: a 4-layer float32
        # stack, 8 x 16 x 32 x 32 in 4 micro-batches over 2 partitions.  A
        # program that checks its pipeline or trains a toy runs this; launches
        # and host work are what it pays.
        _step("tiny-fp32-step", "stack", "fp32", "always", b=2, m=4, n=2, lanes=1, layers=4, c=16,
              h=32, w=32),
        # The headline: partition 1 of 4 of the 5-level U-Net, 32 x 64 x 192 x
        # 192, all 8 micro-batches a call, every one checkpointed.
        _unet_stage("unet-stage", 64, 192, 7, b=4, m=8, group=8, mode="always"),
        # A whole training step of a U-Net on RGB images, with the loss, over
        # 3 partitions and two lanes: decoder, concatenations and the
        # one-channel head are in it.
        _step("unet-rgb-step", "unet", "bf16", "always", b=4, m=4, n=3, lanes=2, levels=3, base=64,
              in_c=3, hw=192),
        # Depthwise / pointwise cells at the size of the 18-cell workload
        # (256 channels, 56 x 56), 16 micro-batches a call.
        _cells("cells-256", 2, 256, 56, 56, b=4, m=16, group=16, mode="except_last"),
        # The same block where the channel count is no power of two and the
        # micro-batch is odd.
        _cells("cells-192", 2, 192, 28, 28, b=3, m=4, group=4, mode="always"),
        # An ordinary hidden layer at an image-network size.
        _layer("conv-56", "conv3", 128, 128, 56, 56, b=8, m=4, group=4),
        # A ragged image and an odd micro-batch, one micro-batch a call, as
        # programs that crop their inputs have it; no ReLU.
        _layer("conv-ragged", "conv3", 128, 192, 45, 61, b=3, m=2, group=1, mode="always",
               relu=False),
        # A thin network's level under a pool: 32 -> 64 channels at 80 x 80.
        _layer("conv-narrow", "conv3", 32, 64, 80, 80, b=4, m=4, group=4, mode="always", pool=True),
        # The deep end of the 6-level U-Net: few pixels, long sums, and
        # weights that outweigh the activations.
        _layer("conv-deep", "conv3", 2048, 2048, 16, 16, b=2, m=2, group=2),
        # A pointwise expansion, a projection without ReLU.
        _layer("pointwise", "conv1", 256, 1024, 28, 28, b=4, m=2, group=2, relu=False),
        # A float32 layer, for programs that train in full precision.
        _layer("conv-fp32", "conv3", 64, 64, 64, 64, b=2, m=2, group=1, mode="always",
               dtype="fp32", relu=False),
        # One image through one layer, forward and backward: latency.
        _layer("conv-b1", "conv3", 64, 64, 56, 56, b=1, m=1, group=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    c = _log(rng, lo, hi)
    step = rng.choice((64, 64, 16, 8)) if c >= 48 else rng.choice((16, 8))
    return max(step, (c + step // 2) // step * step)


def _split(rng):
    m = rng.choice((1, 2, 3, 4, 6, 8))
    return rng.randint(1, 8), m, rng.choice((1, m))


def _draw(rng):
    kind = rng.choice(("conv", "conv", "conv", "conv", "pointwise", "pointwise", "cells", "fp32",
                       "stack", "unet", "unet-stage"))
    mode = rng.choice(sorted(MODES))
    b, m, group = _split(rng)
    h = _log(rng, 8, 224)
    w = h if rng.random() < 0.5 else _log(rng, 8, 224)
    relu = rng.random() < 0.7
    if kind == "conv":
        return _layer(None, "conv3", _channels(rng, 16, 1024), _channels(rng, 16, 1024), h, w, b, m,
                      group, mode, pool=rng.random() < 0.2, relu=relu)
    if kind == "pointwise":
        cout = rng.randint(1, 4) if rng.random() < 0.15 else _channels(rng, 16, 1024)
        return _layer(None, "conv1", _channels(rng, 16, 1024), cout, h, w, b, m, group, mode,
                      relu=relu)
    if kind == "cells":
        h = _log(rng, 7, 112)
        return _cells(None, rng.randint(1, 3), _channels(rng, 32, 512), h, h, b, m, group, mode)
    if kind == "fp32":
        return _layer(None, rng.choice(("conv3", "conv1")), _channels(rng, 8, 128),
                      _channels(rng, 8, 128), _log(rng, 8, 96), _log(rng, 8, 96), rng.randint(1, 4),
                      m, group, mode, dtype="fp32", relu=relu)
    if kind == "stack":
        n = rng.randint(1, 2)
        return _step(None, "stack", "fp32", mode, b=rng.randint(1, 4), m=m, n=n,
                     lanes=rng.choice((1, 2)), layers=rng.randint(2, 5), c=_channels(rng, 8, 32),
                     h=_log(rng, 16, 48), w=_log(rng, 16, 48))
    if kind == "unet":
        levels = rng.randint(2, 3)
        hw = max(1, _log(rng, 32, 192) >> (levels - 1)) << (levels - 1)
        return _step(None, "unet", "bf16", mode, b=rng.randint(1, 4), m=m, n=rng.randint(1, 3),
                     lanes=rng.choice((1, 2)), levels=levels, base=rng.choice((16, 32, 48, 64)),
                     in_c=rng.choice((1, 3, 16, 64)), hw=hw)
    return _unet_stage(None, rng.choice((32, 64, 64)), _log(rng, 4, 24) * 8, rng.randint(2, 4),
                       rng.randint(1, 4), m, group, mode)


def draw(rng):
    """A case of the same ranges.  The caps keep each kind within the listed
    cases' cost, also where the library has only its general kernels for it."""
    caps = {"layer": 1.5e11, "cells": 1e11, "unet-stage": 1.2e12, "unet": 8e11, "stack": 2e10}
    while True:
        c = _draw(rng)
        cap = 3e10 if c["kind"] == "layer" and c["dtype"] == "fp32" else caps[c["kind"]]
        wk = work(c)
        if wk["flops"] <= cap and wk["bytes"] <= 4e9:
            return c


# ---------------------------------------------------------------- networks

def _unet_layers(levels, base, in_c, upto=None):
    ch = [base << l for l in range(levels)]
    out, prev = [], in_c
    for l in range(levels):
        out.append((CONV3, prev, ch[l], 1, 1, POOL if l else NOPRO, -1, -1))
        out.append((CONV3, ch[l], ch[l], 1, 1, NOPRO, l if l < levels - 1 else -1, -1))
        prev = ch[l]
    if upto:
        return out[:upto]
    for l in range(levels - 2, -1, -1):
        out.append((CONV3, prev + ch[l], ch[l], 1, 1, UPCAT, -1, l))
        out.append((CONV3, ch[l], ch[l], 1, 1, NOPRO, -1, -1))
        prev = ch[l]
    out.append((CONV1, prev, 1, 0, 1, NOPRO, -1, -1))
    return out


def _net(case):
    """(layers, in_c, H, W): tuples of tgp_layer, and the input's shape."""
    k = case["kind"]
    if k == "layer":
        op = {"conv3": CONV3, "conv1": CONV1}[case["op"]]
        s = 2 if case["pool"] else 1
        return ([(op, case["cin"], case["cout"], int(case["relu"]), int(case["bias"]),
                  POOL if case["pool"] else NOPRO, -1, -1)], case["cin"], s * case["h"],
                s * case["w"])
    if k == "cells":
        c = case["c"]
        return ([(DW3, c, c, 0, 0, NOPRO, -1, -1), (CONV1, c, c, 1, 1, NOPRO, -1, -1)]
                * case["cells"], c, case["h"], case["w"])
    if k == "unet-stage":   # its stashed outputs are exported skips
        return (_unet_layers(5, case["base"], case["base"], case["layers"]), case["base"],
                case["hw"], case["hw"])
    if k == "stack":
        return ([(CONV3, case["c"], case["c"], 1, 1, NOPRO, -1, -1)] * case["layers"], case["c"],
                case["h"], case["w"])
    return (_unet_layers(case["levels"], case["base"], case["in_c"]), case["in_c"], case["hw"],
            case["hw"])


def _is_step(case):
    return case["kind"] in ("stack", "unet")


def _shapes(layers, H, W):
    out = []
    for l in layers:
        if l[5] == POOL:
            H, W = H // 2, W // 2
        elif l[5] == UPCAT:
            H, W = 2 * H, 2 * W
        out.append((H, W))
    return out


def _wshape(l):
    return (l[1], 9) if l[0] == DW3 else (l[2], 9 if l[0] == CONV3 else 1, l[1])


def _tensors(case, seed):
    """The case's inputs: x, upstream gradients or target, weights, biases."""
    dt = DT[case["dtype"]][1]
    layers, in_c, H, W = _net(case)
    B = case["b"] * case["m"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    x = normal(B, H, W, in_c)
    if case["kind"] in ("layer", "cells"):
        x = x.relu_()
    shapes = _shapes(layers, H, W)
    t = {"x": x.to(dt), "w": [], "b": [], "dskip": {}}
    t["up"] = normal(B, *shapes[-1], layers[-1][2]).to(dt)
    for l, hw in zip(layers, shapes):
        fan = 9 if l[0] == DW3 else (9 if l[0] == CONV3 else 1) * l[1]
        t["w"].append((normal(*_wshape(l)) * math.sqrt(2.0 / fan)).to(dt))
        t["b"].append(normal(l[2]) * 0.1 if l[4] else None)
        if l[6] >= 0 and not _is_step(case):
            t["dskip"][l[6]] = normal(B, *hw, l[2]).to(dt)
    return t


class _State:
    """A program's network: the handle, its parameters, plan and buffers."""

    def __init__(self, case, seed):
        self.case = case
        code = DT[case["dtype"]][0]
        layers, in_c, H, W = _net(case)
        b, m, mode = case["b"], case["m"], MODES[case["mode"]]
        B = b * m
        step = _is_step(case)
        self.t = t = _tensors(case, seed)
        self.h = tgp.net_create(layers, in_c, H, W, code)
        tgp.set_partition(self.h, case["n"] if step else 1)
        self.dw = [torch.zeros(w.shape, device="cuda") for w in t["w"]]
        self.db = [None if v is None else torch.zeros(v.shape, device="cuda") for v in t["b"]]
        for k, (w, v, dw, db) in enumerate(zip(t["w"], t["b"], self.dw, self.db)):
            tgp.bind_params(self.h, k, w.data_ptr(), None if v is None else v.data_ptr(),
                            dw.data_ptr(), None if db is None else db.data_ptr())
        tgp.set_lanes(self.h, case["lanes"] if step else case["group"])
        self.ws = torch.empty(max(256, tgp.plan(self.h, B, m, mode)), dtype=torch.uint8,
                              device="cuda")
        tgp.bind_workspace(self.h, self.ws.data_ptr(), self.ws.numel())
        self.y = torch.empty_like(t["up"])
        self.out = {"y": self.y, "dw": self.dw, "db": [v for v in self.db if v is not None]}
        if step:
            self.loss = torch.zeros(1, device="cuda")
            self.out["loss"] = self.loss
            self.args = (t["x"].data_ptr(), t["up"].data_ptr(), B, m, case["n"], mode,
                         self.loss.data_ptr(), self.y.data_ptr())
            return
        self.dx = torch.empty_like(t["x"])
        self.out["dx"] = self.dx
        self.ckpt = [mode == tgp.CKPT_ALWAYS or (mode == tgp.CKPT_EXCEPT_LAST and i < m)
                     for i in range(1, m + 1)]

        def slices(v):
            return [v.data_ptr() + k * (v.numel() // m) * v.element_size() for k in range(m)]
        self.xs, self.ys, self.dys, self.dxs = (slices(v) for v in (t["x"], self.y, t["up"],
                                                                     self.dx))
        skips = []   # exported skips: read where the library leaves them
        for sid, d in sorted(t["dskip"].items()):
            for i in range(1, m + 1):
                part = d[(i - 1) * b:i * b]
                self._stash(i, sid, True, part).copy_(part)
                skips.append(self._stash(i, sid, False, part))
        if skips:
            self.out["skips"] = skips

    def _stash(self, i, sid, grad, like):
        """Micro-batch i's slot of a skip or its gradient, a view of the workspace."""
        at = tgp.stash_ptr(self.h, i, sid, grad) - self.ws.data_ptr()
        n = like.numel() * like.element_size()
        return self.ws[at:at + n].view(like.dtype).view(like.shape)

    def __del__(self):
        tgp.net_destroy(self.h)


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    if _is_step(s.case):
        tgp.pipeline_step(s.h, *s.args, stream)
        return s.out
    m, g = s.case["m"], s.case["group"]
    if g == 1:
        for i in range(1, m + 1):
            tgp.stage_forward(s.h, 1, i, s.ckpt[i - 1], s.xs[i - 1], s.ys[i - 1], stream)
        for i in range(m, 0, -1):
            tgp.stage_backward_recompute(s.h, 1, i, s.dys[i - 1], s.dxs[i - 1], stream)
            tgp.grad_accumulate(s.h, 1, i, i == m, stream)
        return s.out
    for i in range(1, m + 1, g):
        a = slice(i - 1, i - 1 + g)
        tgp.stage_forward_n(s.h, 1, i, s.ckpt[a], s.xs[a], s.ys[a], stream)
    for i in range(m, 0, -g):
        a = slice(i - g, i)
        tgp.stage_backward_recompute_n(s.h, 1, i, s.dys[a][::-1], s.dxs[a][::-1], stream)
        tgp.grad_accumulate_n(s.h, 1, i, g, i == m, stream)
    return s.out


# ---------------------------------------------------------------- what they need

def work(case):
    """Each tensor the caller hands over or gets read or written once;
    products of the forward, of its repetition where the policy checkpoints,
    and of the two gradients (a pipeline step's first layer has only one)."""
    layers, in_c, H, W = _net(case)
    B, m = case["b"] * case["m"], case["m"]
    esz = 2 if case["dtype"] == "bf16" else 4
    step = _is_step(case)
    again = {"always": 1.0, "except_last": (m - 1) / m, "never": 0.0}[case["mode"]]
    flops = nbytes = 0
    for k, (l, (h, w)) in enumerate(zip(layers, _shapes(layers, H, W))):
        taps = 1 if l[0] == CONV1 else 9
        f = 2 * B * h * w * l[2] * taps * (1 if l[0] == DW3 else l[1])
        flops += f * (1 + again + (1 if step and k == 0 else 2))
        nbytes += math.prod(_wshape(l)) * (esz + 4) + (8 * l[2] if l[4] else 0)
        if l[6] >= 0 and not step:
            nbytes += 2 * B * h * w * l[2] * esz
    h, w = _shapes(layers, H, W)[-1]
    nbytes += B * H * W * in_c * esz * (1 if step else 2) + 2 * B * h * w * layers[-1][2] * esz
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """Between two correct orders of summation.  A stored bf16 value differs
    by 1.7e-3 at most places from the 64-bit one.  Where a pre-activation or
    a pool window's two largest lie within rounding of each other, the two
    orders send a whole gradient element another way: over several layers that
    is what counts (0.016 to 0.039 seen on the U-Nets), and in float32 the one
    such element in a million sets the gradients' 2-norm off by about 1e-3."""
    if case["kind"] in ("unet", "unet-stage", "cells"):
        return {"rel": 0.03, "max": 0.95}
    if case["kind"] == "stack":
        return {"rel": 0.01, "max": 0.5}
    return {"rel": 5e-3, "max": 0.4} if case["dtype"] == "fp32" else {"rel": 0.01, "max": 0.4}


# ---------------------------------------------------------------- in 64 bits

def _taps(l):
    return [(r, s) for r in range(3) for s in range(3)] if l[0] != CONV1 else [(1, 1)]


def _shifted(x, r, s):
    """x moved so that element (h, w) is its neighbour (h + r - 1, w + s - 1)."""
    H, W = x.shape[1:3]
    return torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))[:, r:r + H, s:s + W, :]


def _conv(l, x, w):
    y = 0
    for k, (r, s) in enumerate(_taps(l)):
        v = _shifted(x, r, s)
        y = y + (v * w[:, k] if l[0] == DW3 else (v.reshape(-1, l[1]) @ w[:, k].t().contiguous())
                 .view(*x.shape[:3], l[2]))
    return y


def _conv_dx(l, dz, w):
    dx = 0
    for k, (r, s) in enumerate(_taps(l)):
        v = _shifted(dz, 2 - r, 2 - s)
        dx = dx + (v * w[:, k] if l[0] == DW3 else (v.reshape(-1, l[2]) @ w[:, k])
                   .view(*dz.shape[:3], l[1]))
    return dx


def _conv_dw(l, x, dz):
    out = []
    for r, s in _taps(l):
        v = _shifted(x, r, s)
        if l[0] == DW3:
            out.append((v * dz).sum((0, 1, 2)))
        else:
            out.append(dz.reshape(-1, l[2]).t().contiguous() @ v.reshape(-1, l[1]))
    return torch.stack(out, 1)


def _windows(x):
    n, h, w, c = x.shape
    return x.view(n, h // 2, 2, w // 2, 2, c).permute(0, 1, 3, 5, 2, 4).reshape(
        n, h // 2, w // 2, c, 4)


def exact(case, seed):
    layers, _, _, _ = _net(case)
    t = _tensors(case, seed)
    ws = [w.double() for w in t["w"]]
    step = _is_step(case)
    x, ins, outs, pres, stash, skips = t["x"].double(), [], [], [], {}, []
    for k, l in enumerate(layers):
        pres.append(x)
        if l[5] == POOL:
            x = _windows(x).max(-1).values
        elif l[5] == UPCAT:
            x = torch.cat((x.repeat_interleave(2, 1).repeat_interleave(2, 2), stash[l[7]]), 3)
        ins.append(x)
        x = _conv(l, x, ws[k])
        if l[4]:
            x = x + t["b"][k].double()
        if l[3]:
            x = x.relu()
        outs.append(x)
        if l[6] >= 0:
            stash[l[6]] = x
    y, up = x, t["up"].double()
    out = {"y": y, "dw": [None] * len(layers), "db": []}
    g, gstash = up, {k: v.double() for k, v in t["dskip"].items()}
    if step:
        out["loss"] = ((y - up) ** 2).mean().view(1)
        g = 2 * (y - up) / y.numel()
    for k in range(len(layers) - 1, -1, -1):
        l = layers[k]
        if l[6] >= 0:
            g = g + gstash[l[6]]
        if l[3]:
            g = g * (outs[k] > 0)
        out["dw"][k] = _conv_dw(l, ins[k], g)
        if l[4]:
            out["db"].insert(0, g.sum((0, 1, 2)))
        if k == 0 and step:
            break
        g = _conv_dx(l, g, ws[k])
        if l[5] == POOL:
            v = _windows(pres[k])
            v = torch.nn.functional.one_hot(v.argmax(-1), 4) * g.unsqueeze(-1)
            n, h, w, c, _ = v.shape
            g = v.view(n, h, w, c, 2, 2).permute(0, 1, 4, 2, 5, 3).reshape(n, 2 * h, 2 * w, c)
        elif l[5] == UPCAT:
            c = l[1] - stash[l[7]].shape[3]
            gstash[l[7]] = g[..., c:]
            g = g[..., :c]
            n, h, w, _ = g.shape
            g = g.reshape(n, h // 2, 2, w // 2, 2, c).sum((2, 4))
    if not step:
        out["dx"] = g
    # Gradients that a choice taken on rounded values decides have no such
    # value: three pools leave them 0.1 from those of the unrounded choices;
    # the image layer's sums noise that cancels (up to 0.1 too); and where one
    # float32 pre-activation in a million has the other sign, float32 sums are
    # 1e-4 off with it and 1e-7 without.
    none = [None] * len(layers)
    if case["kind"] == "unet-stage" and len(layers) > 4:
        out.update(dw=none, db=none, dx=None)
    elif case["kind"] == "unet":
        out["dw"][0] = None
    elif case["kind"] == "stack" or (case["kind"] == "layer" and case["relu"]):
        out.update(dw=none, db=none)
        if case["dtype"] == "fp32" and not step:
            out["dx"] = None
    if t["dskip"]:
        b = case["b"]
        out["skips"] = [stash[s][i * b:(i + 1) * b] for s in sorted(t["dskip"])
                        for i in range(case["m"])]
    return out
