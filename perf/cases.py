"""The work that a program using this library has it do, as cases that can be timed and checked.

A case is one pass of such a program through the public entry points of
``paper_1808_05567_amd.conv``:

  fwd     a layer of an inference network: forward with the fused scale / bias / residual /
          ReLU that follows the convolution
  block   a whole residual bottleneck of such a network: three fused forward passes, each
          reading the blocked tensor that the one before it wrote
  step    a layer of a training step: forward, backward by data, weight update
  first   the first layer of a training step, whose input needs no gradient: forward, update
  layout  what stands at the edge of the blocked layout: packing an NCHW tensor, unpacking a
          result

over the ResNet-50 and Inception-v3 layer shapes of ``paper_1808_05567_amd.inputs`` and odd
sizes of the same families, minibatches from 1 (serving) over 28 and 70 (the ones that the
paper trains with) to 256, in fp32 and bf16.
"""
import math

import torch

from paper_1808_05567_amd import conv, inputs

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_CONV = {"f32": conv.CONV_F32, "bf16": conv.CONV_BF16}


def _layer(name, kind, dtype, N, C, K, H, W, R, S, stride, pad_h, pad_w, **more):
    c = {"kind": kind, "dtype": dtype, "N": N, "C": C, "K": K, "H": H, "W": W, "R": R, "S": S,
         "stride": stride, "pad_h": pad_h, "pad_w": pad_w}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # one image through a 3x3 layer of a served network: latency, and few output pixels
        _layer("serve_b1_bf16_3x3_14", "fwd", "bf16", 1, 256, 256, 14, 14, 3, 3, 1, 1, 1,
               scale=True, residual=False, relu=True),
        # one image through the 1x1 layer that closes a residual block, in full precision
        _layer("serve_b1_f32_1x1_7", "fwd", "f32", 1, 512, 2048, 7, 7, 1, 1, 1, 0, 0,
               scale=True, residual=True, relu=True),
        # a served bottleneck block with a small batch of requests
        _layer("serve_b8_bf16_block_14", "block", "bf16", 8, 1024, 256, 14, 14, 3, 3, 1, 1, 1),
        # a batch of requests through a rectangular filter on an odd-sized image
        _layer("serve_b32_bf16_1x7_17", "fwd", "bf16", 32, 192, 192, 17, 17, 1, 7, 1, 0, 3,
               scale=False, residual=False, relu=True),
        # the first layer of a training step, three channels in
        _layer("first_b32_bf16_7x7s2_224", "first", "bf16", 32, 3, 64, 224, 224, 7, 7, 2, 3, 3),
        # training steps at the minibatches of one socket (28), one many-core node (70) and 32
        _layer("step_b28_f32_3x3_28", "step", "f32", 28, 128, 128, 28, 28, 3, 3, 1, 1, 1),
        _layer("step_b70_bf16_1x1_14", "step", "bf16", 70, 1024, 256, 14, 14, 1, 1, 1, 0, 0),
        _layer("step_b32_bf16_3x3_7", "step", "bf16", 32, 512, 512, 7, 7, 3, 3, 1, 1, 1),
        # a grid reduction: unpadded stride-2 3x3 on an odd-sized image
        _layer("step_b32_bf16_3x3s2_35", "step", "bf16", 32, 288, 384, 35, 35, 3, 3, 2, 0, 0),
        # training steps at the benchmark's minibatch: a strided projection in fp32, a wide
        # image in bf16
        _layer("step_b256_f32_1x1s2_28", "step", "f32", 256, 512, 1024, 28, 28, 1, 1, 2, 0, 0),
        _layer("step_b256_bf16_3x3_56", "step", "bf16", 256, 64, 64, 56, 56, 3, 3, 1, 1, 1),
        # an NCHW batch into the blocked layout, and a blocked result back out of it
        _layer("layout_b64_f32_56", "layout", "f32", 64, 64, 256, 56, 56, 1, 1, 1, 0, 0),
    ]


# A drawn case does at most the work of the largest listed ones.
_MOST_FLOPS = 3 * 2 * 256 * 64 * 64 * 56 * 56 * 9
_MOST_BYTES = 1.2e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fwd"] * 6 + ["block"] * 2 + ["step"] * 9 + ["first"] * 2 + ["layout"])
    dtype = rng.choice(["f32", "bf16"])
    N = _log_int(rng, 1, 64) if kind in ("fwd", "block") else _log_int(rng, 8, 256)
    more = {}
    if kind == "first":
        HW = rng.choice([224, 160, 193])
        shape = rng.choice([(3, 64, HW, HW, 7, 7, 2, 3, 3), (3, 32, 299, 299, 3, 3, 2, 0, 0)])
    elif kind == "block":
        width, HW = rng.choice([(64, 56), (128, 28), (256, 14), (512, 7)])
        shape = (4 * width, width, HW, HW, 3, 3, 1, 1, 1)
    else:
        if rng.random() < 0.65:
            t = rng.choice([l for l in inputs.TABLE_I + inputs.INCEPTION_V3 if l.C > 4])
            shape = (t.C, t.K, t.H, t.W, t.R, t.S, t.stride) + t.pads
        else:  # an odd size of the same families
            R, S, stride = rng.choice([(1, 1, 1), (1, 1, 1), (1, 1, 2), (3, 3, 1), (3, 3, 1), (3, 3, 2),
                                       (1, 7, 1), (7, 1, 1)])
            C, K = 4 * _log_int(rng, 8, 192), 4 * _log_int(rng, 8, 192)
            H = _log_int(rng, 7, 60)
            shape = (C, K, H, H + rng.randint(-2, 3), R, S, stride, (R - 1) // 2, (S - 1) // 2)
        if kind == "fwd":
            more = {"scale": rng.random() < 0.5, "residual": rng.random() < 0.4, "relu": rng.random() < 0.8}
    case = _layer(None, kind, dtype, N, *shape, **more)
    while case["N"] > 1:
        w = work(case)
        # (an fp32 operation costs 16 times a bf16 one)
        if w["flops"] * (16 if dtype == "f32" else 1) <= 8 * _MOST_FLOPS and w["flops"] <= _MOST_FLOPS \
                and w["bytes"] <= _MOST_BYTES:
            break
        case["N"] = max(1, case["N"] * 3 // 4)
    return case


# ---------------------------------------------------------------------------
# Inputs: logical tensors from the seed alone.  Activations and gradients uniform on [-1, 1),
# weights normal with standard deviation sqrt(2 / (C R S)), as in the layer benchmark.
# ---------------------------------------------------------------------------
def _extent(c):
    return ((c["H"] + 2 * c["pad_h"] - c["R"]) // c["stride"] + 1,
            (c["W"] + 2 * c["pad_w"] - c["S"]) // c["stride"] + 1)


def _block_layers(c):
    """(C, K, R, S, pad) of the three convolutions of a bottleneck block."""
    return [(c["C"], c["K"], 1, 1, 0), (c["K"], c["K"], c["R"], c["S"], c["pad_h"]),
            (c["K"], c["C"], 1, 1, 0)]


def _logical(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(180805567 + seed)
    dt = _TORCH[c["dtype"]]

    def uniform(*shape):
        return torch.rand(shape, generator=g, device="cuda").mul_(2).sub_(1).to(dt)

    def weights(K, C, R, S):
        return torch.randn((K, C, R, S), generator=g, device="cuda").mul_(math.sqrt(2.0 / (C * R * S))).to(dt)

    def per_channel(K):
        return (torch.rand(K, generator=g, device="cuda") + 0.5, torch.randn(K, generator=g, device="cuda") * 0.1)

    P, Q = _extent(c)
    N, C, K = c["N"], c["C"], c["K"]
    t = {"x": uniform(N, C, c["H"], c["W"])}
    if c["kind"] == "block":
        t["layers"] = [(weights(k, ch, r, s),) + per_channel(k) for ch, k, r, s, _ in _block_layers(c)]
        return t
    if c["kind"] == "layout":
        t["y"] = uniform(N, K, P, Q)
        return t
    t["w"] = weights(K, C, c["R"], c["S"])
    if c["kind"] == "fwd":
        t["scale"], t["bias"] = per_channel(K)
        if c["residual"]:
            t["residual"] = uniform(N, K, P, Q)
    else:
        t["dy"] = uniform(N, K, P, Q)
    return t


class _Plan:
    """A convolution handle, what conv_query says of it, and buffers of the sizes it names."""

    def __init__(self, c, C, K, R, S, stride, pads):
        self.dtype = _TORCH[c["dtype"]]
        self.h = conv.conv_create(c["N"], C, K, c["H"], c["W"], R, S, stride, pads, _CONV[c["dtype"]])
        self.info = conv.conv_query(self.h)
        self.ws = torch.empty(max(16, self.info.workspace_bytes), dtype=torch.uint8, device="cuda")

    def __del__(self):
        if getattr(self, "h", None) is not None:
            conv.conv_destroy(self.h)
            self.h = None

    def _empty(self, nbytes, dtype=None):
        dtype = dtype or self.dtype
        return torch.empty(nbytes // dtype.itemsize, dtype=dtype, device="cuda")

    def input(self):
        return self._empty(self.info.in_bytes)

    def output(self):
        return self._empty(self.info.out_bytes)

    def weights(self, w):
        t = self._empty(self.info.wt_bytes)
        conv.conv_pack_wt(self.h, w, t)
        return t

    def dweights(self):
        return self._empty(self.info.dwt_bytes, torch.float32)

    def packed_input(self, x):
        t = self.input()
        conv.conv_pack_in(self.h, x, t)
        return t

    def packed_output(self, y):
        t = self.output()
        conv.conv_pack_out(self.h, y, t)
        return t

    def channels(self, v):
        t = torch.zeros(self.info.Kp, dtype=torch.float32, device="cuda")
        t[:v.numel()] = v
        return t


def prepare(case, seed):
    c = case
    t = _logical(c, seed)
    st = {"case": c}
    if c["kind"] == "block":
        st["plans"] = plans = [_Plan(c, C, K, R, S, 1, (pad, pad)) for C, K, R, S, pad in _block_layers(c)]
        st["x"] = plans[0].packed_input(t["x"])
        st["layers"] = [(p.weights(w), p.channels(s), p.channels(b)) for p, (w, s, b) in zip(plans, t["layers"])]
        st["outs"] = [p.output() for p in plans]
        return st
    p = st["plan"] = _Plan(c, c["C"], c["K"], c["R"], c["S"], c["stride"], (c["pad_h"], c["pad_w"]))
    if c["kind"] == "layout":
        st["x"], st["y"] = t["x"], p.packed_output(t["y"])
        st["x_blk"], st["y_log"] = p.input(), torch.empty_like(t["y"])
        return st
    st["x"], st["w"], st["y"] = p.packed_input(t["x"]), p.weights(t["w"]), p.output()
    if c["kind"] == "fwd":
        st["scale"] = p.channels(t["scale"]) if c["scale"] else None
        st["bias"] = p.channels(t["bias"])
        st["residual"] = p.packed_output(t["residual"]) if c["residual"] else None
    else:
        st["dy"], st["dw"] = p.packed_output(t["dy"]), p.dweights()
        if c["kind"] == "step":
            st["dx"] = p.input()
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "block":
        x = st["x"]
        for i, (p, (w, s, b), y) in enumerate(zip(st["plans"], st["layers"], st["outs"])):
            conv.conv_fwd_fused_norm(p.h, x, w, y, s, b, st["x"] if i == 2 else None, True, p.ws)
            x = y
        return list(st["outs"])
    p = st["plan"]
    if kind == "layout":
        conv.conv_pack_in(p.h, st["x"], st["x_blk"])
        conv.conv_unpack_out(p.h, st["y"], st["y_log"])
        return {"x_blk": st["x_blk"], "y": st["y_log"]}
    if kind == "fwd":
        conv.conv_fwd_fused_norm(p.h, st["x"], st["w"], st["y"], st["scale"], st["bias"], st["residual"],
                                 c["relu"], p.ws)
        return st["y"]
    conv.conv_fwd(p.h, st["x"], st["w"], st["y"], p.ws)
    out = {"y": st["y"]}
    if kind == "step":
        conv.conv_bwd_data(p.h, st["dy"], st["w"], st["dx"], p.ws)
        out["dx"] = st["dx"]
    conv.conv_upd(p.h, st["x"], st["dy"], st["dw"], p.ws)
    out["dw"] = st["dw"]
    return out


def work(case):
    c = case
    es = 4 if c["dtype"] == "f32" else 2
    P, Q = _extent(c)
    N, C, K = c["N"], c["C"], c["K"]
    if c["kind"] == "block":
        flops = nbytes = 0
        for ch, k, r, s, _ in _block_layers(c):
            flops += 2 * N * k * ch * r * s * c["H"] * c["W"]
            nbytes += es * (N * c["H"] * c["W"] * (ch + k) + k * ch * r * s)
        return {"bytes": nbytes + es * N * C * c["H"] * c["W"], "flops": flops}
    x, y = N * C * c["H"] * c["W"], N * K * P * Q
    if c["kind"] == "layout":
        return {"bytes": 2 * es * (x + y), "flops": 0}
    w = K * C * c["R"] * c["S"]
    # (an unpadded strided 1x1 filter reads only the pixels it samples)
    read = N * C * P * Q if c["R"] * c["S"] == 1 and c["pad_h"] == 0 and c["pad_w"] == 0 else x
    flops = 2 * N * K * C * P * Q * c["R"] * c["S"]
    fwd = es * (read + w + y)
    if c["kind"] == "fwd":
        return {"bytes": fwd + (es * y if c["residual"] else 0), "flops": flops}
    upd = es * (read + y) + 4 * w
    if c["kind"] == "first":
        return {"bytes": fwd + upd, "flops": 2 * flops}
    return {"bytes": fwd + es * (y + w + x) + upd, "flops": 3 * flops}


def tolerance(case):
    if case["kind"] == "layout":
        return "exact"
    if case["dtype"] == "f32":
        # sums of up to 4608 products in 32 bits, dW of up to 2e5 pixels in partial sums: 1e-7 to
        # 6e-7 of the 64-bit result
        return {"rel": 3e-6, "max": 6e-5}
    # a 32-bit sum rounded once to 8 bits: 1.65e-3 of the 64-bit result, an ulp (2^-7) where a
    # rounding falls the other way; in a block the roundings of two layers travel on
    if case["kind"] == "block":
        return {"rel": 1e-2, "max": 1e-1}
    return {"rel": 6e-3, "max": 2e-2}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch: one matrix product per filter tap.
# ---------------------------------------------------------------------------
def _blocked(t, v):
    """[N][C][H][W] -> [N][Cb][H][W][v], flat."""
    N, C, H, W = t.shape
    Cb = -(-C // v)
    t = torch.nn.functional.pad(t, (0, 0, 0, 0, 0, Cb * v - C))
    return t.reshape(N, Cb, v, H, W).permute(0, 1, 3, 4, 2).contiguous().reshape(-1)


def _blocked_weights(t, v):
    """[K][C][R][S] -> [Cb][R][S][Kp][v], flat."""
    K, C, R, S = t.shape
    Cb, Kp = -(-C // v), -(-K // v) * v
    t = torch.nn.functional.pad(t, (0, 0, 0, 0, 0, Cb * v - C, 0, Kp - K))
    return t.reshape(Kp, Cb, v, R, S).permute(1, 3, 4, 0, 2).contiguous().reshape(-1)


def _taps(x, R, S, stride, pads, P, Q):
    """The input pixels under each tap of the filter: (r, s, [N][C][P*Q])."""
    x = torch.nn.functional.pad(x, (pads[1], pads[1], pads[0], pads[0]))
    for r in range(R):
        for s in range(S):
            v = x[:, :, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride]
            yield r, s, v.reshape(v.shape[0], v.shape[1], P * Q)


def _fwd64(x, w, stride, pads, P, Q):
    y = torch.zeros((x.shape[0], w.shape[0], P * Q), dtype=torch.float64, device=x.device)
    for r, s, v in _taps(x, w.shape[2], w.shape[3], stride, pads, P, Q):
        wt = w[:, :, r, s].contiguous()
        for n in range(x.shape[0]):
            y[n].addmm_(wt, v[n].contiguous())
    return y.reshape(x.shape[0], w.shape[0], P, Q)


def _bwd64(dy, w, H, W, stride, pads):
    N, K, P, Q = dy.shape
    C, R, S = w.shape[1:]
    dx = torch.zeros((N, C, H + 2 * pads[0], W + 2 * pads[1]), dtype=torch.float64, device=dy.device)
    for r in range(R):
        for s in range(S):
            wt = w[:, :, r, s].t().contiguous()
            for n in range(N):
                dx[n, :, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride] += \
                    torch.mm(wt, dy[n].reshape(K, P * Q)).reshape(C, P, Q)
    return dx[:, :, pads[0]:pads[0] + H, pads[1]:pads[1] + W]


def _upd64(x, dy, R, S, stride, pads):
    N, K, P, Q = dy.shape
    dw = torch.zeros((K, x.shape[1], R, S), dtype=torch.float64, device=x.device)
    g = dy.reshape(N, K, P * Q).permute(1, 0, 2).reshape(K, N * P * Q)
    for r, s, v in _taps(x, R, S, stride, pads, P, Q):
        dw[:, :, r, s] = torch.mm(g, v.permute(0, 2, 1).reshape(N * P * Q, x.shape[1]))
    return dw


def exact(case, seed):
    c = case
    if c["kind"] == "layout":
        return None  # whole bytes, compared as they are
    t = _logical(c, seed)
    v = 4 if c["dtype"] == "f32" else 8
    x = t["x"].double()
    pads = (c["pad_h"], c["pad_w"])
    P, Q = _extent(c)
    if c["kind"] == "block":
        outs, a = [], x
        for i, ((w, s, b), (C, K, R, S, pad)) in enumerate(zip(t["layers"], _block_layers(c))):
            y = _fwd64(a, w.double(), 1, (pad, pad), c["H"], c["W"])
            y = y * s.double()[:, None, None] + b.double()[:, None, None]
            a = torch.relu(y + x if i == 2 else y)
            outs.append(_blocked(a, v))
        return outs
    w = t["w"].double()
    y = _fwd64(x, w, c["stride"], pads, P, Q)
    if c["kind"] == "fwd":
        if c["scale"]:
            y = y * t["scale"].double()[:, None, None]
        y = y + t["bias"].double()[:, None, None]
        if c["residual"]:
            y = y + t["residual"].double()
        return _blocked(torch.relu(y) if c["relu"] else y, v)
    out = {"y": _blocked(y, v)}
    del y
    dy = t["dy"].double()
    if c["kind"] == "step":
        out["dx"] = _blocked(_bwd64(dy, w, c["H"], c["W"], c["stride"], pads), v)
    out["dw"] = _blocked_weights(_upd64(x, dy, c["R"], c["S"], c["stride"], pads), v)
    return out
