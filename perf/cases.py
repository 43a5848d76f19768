"""The calls whose speed matters to a program built on this library, over the sizes it is used at.

Every case goes through the Python binding as a program would call it: weights are prepared
once, outputs go to a buffer the program keeps, and each pass takes the activations it is
handed.  All results are whole numbers, so every comparison is exact.

Routes of a 2-D convolution ("kind": "conv"):
  bytes    8-bit activations are packed, then convolved (the benchmark's step: pack, spread, multiply)
  packed   the activations are already in the packed format (temporary spacer bits)
  spaced   the activations are already in the permanent-spacer layout
"""
import math

import torch

import paper_1809_10572_amd as samd

SHAPE_KEYS = ("N", "C", "H", "W", "M", "KH", "KW", "sh", "sw", "ph", "pw")


def _conv(name, shape, xb, xs, wb, route, ends=False):
    c = {"name": name, "kind": "conv", "route": route, "xb": xb, "xs": xs, "wb": wb, "ws": True, "ends": ends}
    c.update(zip(SHAPE_KEYS, shape))
    return c


def _int8(name, shape, xs):
    c = {"name": name, "kind": "int8", "xs": xs}
    c.update(zip(SHAPE_KEYS, shape))
    return c


def listed():
    return [
        # one small layer of a small image: a call bound by launches and by the host
        _conv("single_u4", (1, 16, 16, 16, 16, 3, 3, 1, 1, 1, 1), 4, False, 4, "packed"),
        # the benchmark's layer at its low, middle and high bit widths, from 8-bit activations as its step runs it
        _conv("mid_u2", (8, 128, 56, 56, 128, 3, 3, 1, 1, 1, 1), 2, False, 2, "bytes"),
        _conv("mid_u4", (8, 128, 56, 56, 128, 3, 3, 1, 1, 1, 1), 4, False, 4, "bytes"),
        _conv("mid_u8", (8, 128, 56, 56, 128, 3, 3, 1, 1, 1, 1), 8, False, 8, "bytes"),
        # VGG-B layer 2, signed 8-bit, one image: wide rows, more words to a row than a wave has lanes
        _conv("vggb2_s8", (1, 64, 224, 224, 64, 3, 3, 1, 1, 1, 1), 8, True, 8, "packed"),
        # VGG-B layer 8 in the permanent-spacer layout at a low width: a late, channel-heavy layer
        _conv("vggb8_s3_spaced", (1, 512, 28, 28, 512, 3, 3, 1, 1, 1, 1), 3, True, 3, "spaced"),
        # the AlexNet-shaped stack's first layer: an 11x11 kernel at stride 4 on three channels
        _conv("alex1_u4", (16, 3, 224, 224, 96, 11, 11, 4, 4, 2, 2), 4, False, 4, "packed"),
        # odd sizes everywhere, a 5x5 kernel, operands of different widths, half of the values at the range ends
        _conv("ragged_5x5", (3, 37, 61, 45, 50, 5, 5, 1, 1, 2, 2), 6, True, 5, "packed", True),
        # a whole forward pass of the AlexNet-shaped stack, requantised between layers straight into operand words
        {"name": "stack_u4", "kind": "stack", "bits": 4, "N": 16, "side": 224},
        # the standalone 1-D convolution on 2^20 values
        {"name": "conv1d_2p20", "kind": "conv1d", "n": 1 << 20, "bits": 3, "K": 5},
        # what stands between two layers: the maximum of the stack's largest accumulators, then ReLU and requantisation
        {"name": "requant_55", "kind": "requant", "N": 16, "C": 384, "H": 55, "W": 55, "bits": 4},
        # the native 8-bit path on the stack's third layer
        _int8("int8_alex3", (16, 256, 55, 55, 384, 3, 3, 1, 1, 1, 1), False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, most):
    """A layer of 1x1, 3x3 or 5x5 kernels, some of stride 2, of at most `most` multiply-accumulates."""
    while True:
        k = rng.choice((1, 3, 3, 3, 5))
        s = rng.choice((1, 1, 1, 2))
        shape = (_log(rng, 1, 16), _log(rng, 3, 512), _log(rng, 7, 224), _log(rng, 7, 224), _log(rng, 8, 512), k, k, s, s, k // 2, k // 2)
        if 5e5 <= _macs(dict(zip(SHAPE_KEYS, shape))) <= most:
            return shape


def draw(rng):
    kind = rng.choice(("conv",) * 7 + ("stack", "conv1d", "requant", "int8", "int8"))
    if kind == "conv":
        xb = rng.randint(1, 8)
        wb = xb if rng.random() < 0.7 else rng.randint(1, 8)
        c = _conv("", _shape(rng, 4e9), xb, rng.random() < 0.5, wb, rng.choice(("bytes", "packed", "spaced")), rng.random() < 0.3)
    elif kind == "int8":
        c = _int8("", _shape(rng, 4e10), rng.random() < 0.5)
    elif kind == "stack":
        c = {"kind": "stack", "bits": rng.randint(2, 8), "N": rng.randint(1, 7), "side": rng.randint(64, 224)}
    elif kind == "conv1d":
        c = {"kind": "conv1d", "n": _log(rng, 1 << 12, 1 << 22), "bits": rng.randint(1, 8), "K": rng.choice((2, 3, 4, 5, 7))}
    else:
        c = {"kind": "requant", "N": _log(rng, 1, 16), "C": _log(rng, 8, 384), "H": _log(rng, 7, 112), "W": _log(rng, 7, 55), "bits": rng.randint(1, 8)}
    c.pop("name", None)
    return c


# --- the layers of a case -----------------------------------------------------------------------

def _tuple(c):
    return tuple(c[k] for k in SHAPE_KEYS)


def _out_hw(shape):
    _, _, H, W, _, KH, KW, sh, sw, ph, pw = shape
    return (H + 2 * ph - KH) // sh + 1, (W + 2 * pw - KW) // sw + 1


def _macs(c):
    shape = _tuple(c)
    Ho, Wo = _out_hw(shape)
    return c["N"] * c["C"] * c["M"] * c["KH"] * c["KW"] * Ho * Wo


def _stack_layers(c):
    """The AlexNet-shaped stack on N images of side x side: five layers, no pooling."""
    n, side = c["N"], c["side"]
    s = (side + 4 - 11) // 4 + 1
    return [(n, 3, side, side, 96, 11, 11, 4, 4, 2, 2), (n, 96, s, s, 256, 5, 5, 1, 1, 2, 2), (n, 256, s, s, 384, 3, 3, 1, 1, 1, 1),
            (n, 384, s, s, 384, 3, 3, 1, 1, 1, 1), (n, 384, s, s, 256, 3, 3, 1, 1, 1, 1)]


# --- inputs -------------------------------------------------------------------------------------

def _values(g, shape, bits, signed, ends=False):
    """Uniform over the b-bit range; `ends`: half of the values at the range's two ends."""
    lo, hi = (-(1 << (bits - 1)), (1 << (bits - 1)) - 1) if signed else (0, (1 << bits) - 1)
    dtype = torch.int8 if signed else torch.uint8
    v = torch.randint(lo, hi + 1, shape, generator=g, device=g.device, dtype=torch.int16)
    if ends:
        pick = torch.randint(0, 4, shape, generator=g, device=g.device, dtype=torch.uint8)
        v = torch.where(pick == 0, lo, torch.where(pick == 1, hi, v))
    return v.to(dtype)


def _raw(case, seed):
    """The plain values of a case: what prepare() and exact() both start from."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    kind = case["kind"]
    if kind in ("conv", "int8"):
        n, ch, h, w, m, kh, kw = _tuple(case)[:7]
        xb, wb, ends = case.get("xb", 8), case.get("wb", 8), case.get("ends", False)
        return {"x": _values(g, (n, ch, h, w), xb, case["xs"], ends), "w": _values(g, (m, ch, kh, kw), wb, True, ends)}
    if kind == "stack":
        layers, b = _stack_layers(case), case["bits"]
        return {"x": _values(g, layers[0][:4], b, False), "w": [_values(g, (s[4], s[1], s[5], s[6]), b, True) for s in layers]}
    if kind == "conv1d":
        return {"x": _values(g, (case["n"],), case["bits"], False), "taps": _values(g, (case["K"],), case["bits"], False).tolist()}
    # accumulators of a layer: sums of many products, near normal around zero
    acc = torch.randn((case["N"], case["C"], case["H"], case["W"]), generator=g, device=g.device) * 3000.0
    return {"acc": acc.round().to(torch.int32)}


def _y(shape):
    return torch.empty((shape[0], shape[4]) + _out_hw(shape), dtype=torch.int32, device="cuda")


def prepare(case, seed):
    raw, kind = _raw(case, seed), case["kind"]
    s = {"kind": kind}
    if kind == "conv":
        shape, xf, wf = _tuple(case), samd.Fmt(case["xb"], case["xs"]), samd.Fmt(case["wb"], True)
        wp = samd.pack(raw["w"], wf.bits, True)
        s.update(route=case["route"], shape=shape, xf=xf, wf=wf, y=_y(shape))
        if case["route"] == "spaced":
            s["ws"] = samd.conv2d_spaced_prepare(wp, wf, shape, xf)
            s["x"] = samd.conv2d_spaced_pack(raw["x"], xf, wf, shape)
        else:
            s["ws"] = samd.conv2d_prepare(wp, wf, shape, xf)
            s["x"] = raw["x"] if case["route"] == "bytes" else samd.pack(raw["x"], xf.bits, case["xs"])
    elif kind == "int8":
        shape, xf, wf = _tuple(case), samd.Fmt(8, case["xs"]), samd.Fmt(8, True)
        s.update(shape=shape, xf=xf, wf=wf, y=_y(shape), ws=samd.conv2d_int8_prepare(raw["w"], wf, shape, xf),
                 x=raw["x"].permute(0, 2, 3, 1).contiguous())
    elif kind == "stack":
        layers, b = _stack_layers(case), case["bits"]
        xf, wf = samd.Fmt(b, False), samd.Fmt(b, True)
        s.update(layers=layers, bits=b, xf=xf, wf=wf, x=samd.pack(raw["x"], b, False), y=[_y(l) for l in layers],
                 ws=[samd.conv2d_prepare(samd.pack(w, b, True), wf, l, xf) for w, l in zip(raw["w"], layers)])
    elif kind == "conv1d":
        n, b, K = case["n"], case["bits"], case["K"]
        s.update(n=n, bits=b, taps=raw["taps"], x=samd.pack(raw["x"].view(1, n), b, False).view(-1),
                 y=torch.empty(n - K + 1, dtype=torch.int32, device="cuda"))
    else:
        s.update(acc=raw["acc"], bits=case["bits"], max=torch.empty(1, dtype=torch.int32, device="cuda"),
                 shift=torch.empty(1, dtype=torch.int32, device="cuda"))
    return s


# --- one pass -----------------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "conv":
        if s["route"] == "spaced":
            return samd.conv2d_spaced(s["x"], s["xf"], s["wf"], s["shape"], s["ws"], out=s["y"])
        x = samd.pack(s["x"], s["xf"].bits, bool(s["xf"].is_signed)) if s["route"] == "bytes" else s["x"]
        return samd.conv2d_prepared(x, s["xf"], s["wf"], s["shape"], s["ws"], out=s["y"])
    if kind == "int8":
        return samd.conv2d_int8_prepared(s["x"], s["xf"], s["wf"], s["shape"], s["ws"], out=s["y"])
    if kind == "stack":
        y = samd.conv2d_prepared(s["x"], s["xf"], s["wf"], s["layers"][0], s["ws"][0], out=s["y"][0])
        for i in range(1, len(s["layers"])):
            samd.relu_requant_stage(y, samd.max_i32(y), s["bits"], s["wf"], s["layers"][i], s["ws"][i])
            y = samd.conv2d_accumulate(s["xf"], s["wf"], s["layers"][i], s["ws"][i], out=s["y"][i])
        return y
    if kind == "conv1d":
        return samd.conv1d(s["x"], s["n"], s["bits"], s["taps"], s["bits"], out=s["y"])
    mx = samd.max_i32(s["acc"], out=s["max"])
    return {"max": mx, "packed": samd.relu_requant_pack(s["acc"], mx, s["bits"], shift_out=s["shift"]), "shift": s["shift"]}


# --- what one pass cannot do without ------------------------------------------------------------

def _conv_work(c, x_bits, w_bits):
    shape = _tuple(c)
    Ho, Wo = _out_hw(shape)
    n, ch, h, w, m, kh, kw = shape[:7]
    return {"bytes": n * ch * h * w * x_bits / 8 + m * ch * kh * kw * w_bits / 8 + 4.0 * n * m * Ho * Wo, "flops": 2.0 * _macs(c)}


def work(case):
    kind = case["kind"]
    if kind == "conv":
        return _conv_work(case, 8 if case["route"] == "bytes" else case["xb"], case["wb"])
    if kind == "int8":
        return _conv_work(case, 8, 8)
    if kind == "stack":
        each = [_conv_work(dict(zip(SHAPE_KEYS, l)), case["bits"], case["bits"]) for l in _stack_layers(case)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    if kind == "conv1d":
        outs = case["n"] - case["K"] + 1
        return {"bytes": case["n"] * case["bits"] / 8 + 4.0 * outs, "flops": 2.0 * outs * case["K"]}
    n = case["N"] * case["C"] * case["H"] * case["W"]
    return {"bytes": 4.0 * n + n * case["bits"] / 8, "flops": 2.0 * n}


def tolerance(case):
    return "exact"   # whole numbers throughout


# --- the definition, in 64 bits -----------------------------------------------------------------

def _conv64(x, w, shape):
    """Cross-correlation with zero padding; float64 holds every sum exactly (all are below 2^31)."""
    _, _, _, _, m, kh, kw, sh, sw, ph, pw = shape
    Ho, Wo = _out_hw(shape)
    wm = w.double().reshape(m, -1)
    out = torch.empty((x.shape[0], m, Ho, Wo), dtype=torch.int64, device=x.device)
    for i in range(x.shape[0]):
        cols = torch.nn.functional.unfold(x[i:i + 1].double(), (kh, kw), padding=(ph, pw), stride=(sh, sw))[0]
        out[i] = (wm @ cols).round().to(torch.int64).view(m, Ho, Wo)
    return out


def _requant64(acc, bits):
    """ReLU, then the smallest shift that brings the maximum into b bits, rounding half up; and that shift."""
    r = acc.clamp(min=0)
    shift = max(0, int(r.max()).bit_length() - bits)
    half = (1 << (shift - 1)) if shift else 0
    return ((r + half) >> shift).clamp(max=(1 << bits) - 1), shift


def _pack64(v, bits):
    """Rows of unsigned b-bit values as the packed format's 32-bit words."""
    per = 32 // bits
    width = -(-v.shape[-1] // per) * per
    v = torch.nn.functional.pad(v, (0, width - v.shape[-1]))
    word = (v.view(*v.shape[:-1], width // per, per) << (torch.arange(per, device=v.device) * bits)).sum(-1)
    return torch.where(word >= 1 << 31, word - (1 << 32), word)


def exact(case, seed):
    raw, kind = _raw(case, seed), case["kind"]
    if kind in ("conv", "int8"):
        return _conv64(raw["x"], raw["w"], _tuple(case))
    if kind == "stack":
        layers = _stack_layers(case)
        x = raw["x"]
        for i, l in enumerate(layers):
            y = _conv64(x, raw["w"][i], l)
            if i + 1 < len(layers):
                x = _requant64(y, case["bits"])[0]
        return y
    if kind == "conv1d":
        x, taps = raw["x"].to(torch.int64), raw["taps"]
        outs = case["n"] - case["K"] + 1
        return sum(t * x[case["K"] - 1 - i:case["K"] - 1 - i + outs] for i, t in enumerate(taps))
    acc = raw["acc"].to(torch.int64)
    q, shift = _requant64(acc, case["bits"])
    return {"max": acc.max().view(1), "packed": _pack64(q, case["bits"]), "shift": torch.tensor([shift], device=acc.device)}
