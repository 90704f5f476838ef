"""Workloads whose speed this library answers for, and the values they must give.

Every case is one pass through the public entry points of
``paper_2609_21849_amd`` as a program that serves the denoising transformer,
or its small text encoder, calls them: activations arrive as bf16 tensors,
weights were quantized and packed beforehand. Shapes are those of ``synth``
(hidden 3072, FFN 9216, 4608 tokens for a 1024 x 1024 image; text encoder
hidden 1024, FFN 3072) and ragged sizes between and below them.

Kinds of case:
  linear   one linear layer, Y = X W^T: the activation quantizer (dynamic,
           or static with a calibrated scale) and the GEMM; weight-only
           layers take the bf16 activation as it is. "slice": X is the last
           third of the columns of a three times wider tensor (a projection
           that reads V out of a fused QKV output).
  fused    the few-token FP8 linear that quantizes inside the GEMM.
  block    the four linears of one transformer block with calibrated scales:
           QKV and attention-out write quantized outputs, attention (not a
           part of this library) is stood in for by its V input, GELU is
           torch's.
  weights  offline weight preparation: quantize, pack, and read back as a
           checking tool does (unpack, dequantize).
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

import paper_2609_21849_amd as q

FORMATS = {"fp8": q.QG_FMT_FP8_E4M3, "nvfp4": q.QG_FMT_NVFP4, "mxfp4": q.QG_FMT_MXFP4, "mxfp8": q.QG_FMT_MXFP8,
           "w4a16": q.QG_FMT_NVFP4}
HIDDEN, FFN = 3072, 9216
POOL_N = 355 * 1024  # encoder weights stacked along N: more than twice the 256 MB last-level cache


def _linear(name, fmt, m, n, k, slice_=False, static=False, out="bf16", heavy=False):
    case = {"kind": "linear", "fmt": fmt, "m": m, "n": n, "k": k, "slice": slice_, "static": static, "out": out,
            "heavy": heavy}
    return case if name is None else {"name": name, **case}


def listed():
    return [
        # the smallest call: a modulation-sized linear on a short sequence, one launch
        {"name": "fused_fp8_128x256x256", "kind": "fused", "m": 128, "n": 256, "k": 256, "out": "bf16"},
        # text encoder, one token at a time (decode), weight-only 4 bit
        _linear("w4a16_1x3072x1024", "w4a16", 1, 3072, 1024),
        # text encoder over a prompt of ragged length (prefill), weight-only 4 bit
        _linear("w4a16_300x1024x3072", "w4a16", 300, 1024, 3072),
        # the same encoder with 8-bit weights and activations, a full prompt
        _linear("fp8_256x3072x1024", "fp8", 256, 3072, 1024),
        # text tokens through a transformer linear, 4-bit weights and activations
        _linear("nvfp4_512x3072x3072", "nvfp4", 512, 3072, 3072),
        # the same in the block format the matrix cores read natively, ragged length
        _linear("mxfp4_500x3072x3072", "mxfp4", 500, 3072, 3072),
        # attention-out of a 1024 x 1024 image, reading V in place from the fused QKV output
        _linear("fp8_v_slice_4608x3072x3072", "fp8", 4608, 3072, 3072, slice_=True),
        # MLP-down of the same image in 4 bits, activations with outlier channels
        _linear("nvfp4_4608x3072x9216", "nvfp4", 4608, 3072, 9216, heavy=True),
        # MLP-up of a smaller, ragged image (about 768 x 768 and its text), MX 8 bit
        _linear("mxfp8_2800x9216x3072", "mxfp8", 2800, 9216, 3072),
        # a batch of 16 tokens against weights far larger than the caches
        _linear("w4a16_pool_16", "w4a16", 16, POOL_N, 3072),
        # a whole transformer block of a 1024 x 1024 image, calibrated FP8
        {"name": "block_fp8_4608", "kind": "block", "fmt": "fp8", "m": 4608},
        # preparing one MLP-up weight in 4 bits, once per model and precision
        {"name": "weights_nvfp4_9216x3072", "kind": "weights", "fmt": "nvfp4", "n": 9216, "k": 3072, "out": "bf16"},
    ]


def _log(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choices(["linear", "fused", "block", "weights", "pool"], [70, 8, 6, 8, 8])[0]
    if kind == "fused":
        while True:
            m, k = _log(rng, 1, 256), _log(rng, 128, 3072, 128)
            if m * k <= 65536:  # what the one-launch entry point takes
                return {"kind": "fused", "m": m, "n": _log(rng, 64, 3072, 16), "k": k, "out": rng.choice(["bf16", "f32"])}
    if kind == "block":
        return {"kind": "block", "fmt": rng.choice(["fp8", "nvfp4"]), "m": _log(rng, 256, 2816)}
    if kind == "weights":
        return {"kind": "weights", "fmt": rng.choice(["fp8", "nvfp4", "mxfp4", "mxfp8"]), "n": _log(rng, 256, 9216, 16),
                "k": _log(rng, 256, 9216, 256), "out": rng.choice(["bf16", "f32"])}
    if kind == "pool":
        return _linear(None, "w4a16", rng.randint(1, 16), 1024 * rng.randint(96, 355), rng.choice([1024, 2048, 3072]))
    fmt = rng.choice(["fp8", "nvfp4", "mxfp4", "mxfp8", "w4a16"])
    while True:
        m, n = _log(rng, 1, 4608), _log(rng, 256, 9216, 16)
        k = _log(rng, 256, 9216, 256 if fmt[:2] == "mx" else 128)
        if m * n * k <= 4608 * 9216 * 3072:
            break
    return _linear(None, fmt, m, n, k, slice_=fmt != "w4a16" and rng.random() < 0.25,
                   static=fmt in ("fp8", "nvfp4") and rng.random() < 0.25,
                   out="f32" if rng.random() < 0.2 else "bf16", heavy=rng.random() < 0.25)


# ---------------------------------------------------------------- inputs
def _normal(gen, rows, cols, sigma):
    t = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    step = max(1, (1 << 27) // cols)  # the wide pool in pieces
    for r in range(0, rows, step):
        c = min(step, rows - r)
        t[r:r + c] = sigma * torch.randn((c, cols), generator=gen, device="cuda")
    return t


def _activation(case, gen, m, k, slice_=False, heavy=False):
    x = _normal(gen, m, 3 * k if slice_ else k, 1.0)
    if heavy:  # 0.1 % of the input channels carry outliers, the same ones in every row
        ch = torch.randperm(x.shape[1], generator=gen, device="cuda")[:max(1, round(x.shape[1] / 1000))]
        x[:, ch] *= 50.0
    return x[:, 2 * k:] if slice_ else x


def _inputs(case, seed):
    """The bf16 tensors a case starts from: activation and weights."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000003 + 17)
    kind = case["kind"]
    if kind == "weights":
        return None, {"w": _normal(gen, case["n"], case["k"], 0.02)}
    if kind == "block":
        x = _activation(case, gen, case["m"], HIDDEN)
        shapes = {"qkv": (3 * HIDDEN, HIDDEN), "attn_out": (HIDDEN, HIDDEN), "mlp_up": (FFN, HIDDEN),
                  "mlp_down": (HIDDEN, FFN)}
        return x, {name: _normal(gen, n, k, 0.02) for name, (n, k) in shapes.items()}
    x = _activation(case, gen, case["m"], case["k"], case.get("slice", False), case.get("heavy", False))
    return x, {"w": _normal(gen, case["n"], case["k"], 0.02)}


def _static_scale(case, stage="x"):
    """Calibrated tensor scales: fixed numbers from other data of the same
    distributions (an absolute maximum near the largest value seen)."""
    amax = {"x": 5.25 * (50.0 if case.get("heavy") else 1.0), "v": 5.5, "a": 6.0, "u": 6.5}[stage]
    return torch.tensor([amax / (448.0 if case["fmt"] == "fp8" else 2688.0)], dtype=torch.float32, device="cuda")


def prepare(case, seed):
    x, w = _inputs(case, seed)
    if case["kind"] == "weights":
        return {"case": case, "w": w["w"]}
    fmt = q.QG_FMT_FP8_E4M3 if case["kind"] == "fused" else FORMATS[case["fmt"]]
    state = {"case": case, "fmt": fmt, "x": x, "packed": {name: q.pack(q.quantize(t, fmt)) for name, t in w.items()}}
    if case["kind"] == "block":
        state["scales"] = {s: _static_scale(case, s) for s in ("x", "v", "a", "u")}
    elif case.get("static"):
        state["scale"] = _static_scale(case)
    return state


# ---------------------------------------------------------------- one pass
def _out(case):
    return q.QG_OUT_F32 if case["out"] == "f32" else q.QG_OUT_BF16


def _run_block(s):
    """QKV and attention-out leave quantized tensors; attention-out reads the V
    third of the QKV codes in place."""
    fmt, pk, sc, m = s["fmt"], s["packed"], s["scales"], s["case"]["m"]
    x = q.quantize(s["x"], fmt, static_scale=sc["x"])
    if fmt == q.QG_FMT_FP8_E4M3:
        h = q.linear_fp8_out(x, pk["qkv"], fmt, 3 * HIDDEN, sc["v"])
        a = q.QTensor(fmt, torch.empty((m, HIDDEN), dtype=torch.uint8, device="cuda"), None, sc["a"], m, HIDDEN)
        w = pk["attn_out"]
        q.qg_gemm_quant(fmt, h.codes.data_ptr() + 2 * HIDDEN, None, sc["v"], 3 * HIDDEN, fmt, w, w.numel(), m, HIDDEN,
                        HIDDEN, a.codes, HIDDEN, sc["a"])
    else:
        h = q.linear_nvfp4_out(x, pk["qkv"], fmt, 3 * HIDDEN, sc["v"])
        a = q.QTensor(fmt, torch.empty((m, HIDDEN // 2), dtype=torch.uint8, device="cuda"),
                      torch.empty((m, HIDDEN // 16), dtype=torch.uint8, device="cuda"), sc["a"], m, HIDDEN)
        w = pk["attn_out"]
        q.qg_gemm_quant_nvfp4(fmt, h.codes.data_ptr() + HIDDEN, h.block_scales.data_ptr() + 2 * HIDDEN // 16, sc["v"],
                              3 * HIDDEN, fmt, w, w.numel(), m, HIDDEN, HIDDEN, a.codes, a.block_scales, HIDDEN, sc["a"])
    u = q.linear(a, pk["mlp_up"], fmt, FFN)
    g = q.quantize(F.gelu(u, approximate="tanh"), fmt, static_scale=sc["u"])
    y = q.linear(g, pk["mlp_down"], fmt, HIDDEN)
    return {"qkv_codes": h.codes, "attn_out_codes": a.codes, "mlp_up": u, "y": y}


def run(state):
    case = state["case"]
    if case["kind"] == "block":
        return _run_block(state)
    if case["kind"] == "fused":
        y, scale = q.linear_fp8(state["x"], state["packed"]["w"], case["n"], out_dtype=_out(case))
        return {"y": y, "scale": scale}
    if case["kind"] == "weights":
        fmt = FORMATS[case["fmt"]]
        t = q.quantize(state["w"], fmt)
        back = q.unpack(q.pack(t), fmt, case["n"], case["k"])
        out = {"codes": back.codes, "w": q.dequantize(back, out_dtype=_out(case))}
        if back.block_scales is not None:
            out["block_scales"] = back.block_scales
        return out
    x, fmt = state["x"], state["fmt"]
    a = x if case["fmt"] == "w4a16" else q.quantize(x, fmt, static_scale=state.get("scale"))
    return {"y": q.linear(a, state["packed"]["w"], fmt, case["n"], out_dtype=_out(case))}


# ---------------------------------------------------------------- what a pass cannot do without
def _weight_bits(fmt):
    return {"fp8": 8.0, "nvfp4": 4.5, "w4a16": 4.5, "mxfp4": 4.25, "mxfp8": 8.25}[fmt]


def work(case):
    kind = case["kind"]
    if kind == "weights":
        e = case["n"] * case["k"]
        bits = _weight_bits(case["fmt"])
        # read bf16; write the packed weight, the codes read back and the dequantized weight
        return {"bytes": e * (2 + 2 * bits / 8 + (4 if case["out"] == "f32" else 2)), "flops": 0}
    if kind == "block":
        m, bits = case["m"], _weight_bits(case["fmt"])
        elements = HIDDEN * (3 * HIDDEN + HIDDEN + 2 * FFN)
        act = m * (2 * HIDDEN + (3 * HIDDEN + HIDDEN) * bits / 8 + 2 * FFN + 2 * HIDDEN)
        return {"bytes": elements * bits / 8 + act, "flops": 2.0 * m * elements}
    m, n, k = case["m"], case["n"], case["k"]
    bits = 8.0 if kind == "fused" else _weight_bits(case["fmt"])
    return {"bytes": 2.0 * m * k + n * k * bits / 8 + m * n * (4 if case["out"] == "f32" else 2), "flops": 2.0 * m * n * k}


# ---------------------------------------------------------------- the same in 64 bits
def _f32(v):
    """One correctly rounded fp32 step of a value computed in 64 bits."""
    return v.float().double()


def _e4m3(v):
    return v.float().clamp(-448.0, 448.0).to(torch.float8_e4m3fn).double()


def _e2m1(v):
    a = v.abs()
    c = ((a > 0.25).int() + (a >= 0.75) + (a > 1.25) + (a >= 1.75) + (a > 2.5) + (a >= 3.5) + (a > 5.0))
    grid = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], dtype=torch.float64, device=v.device)
    return torch.copysign(grid[c.long()], v)


def _quantized(x, fmt, scale=None):
    """(codes decoded with their block scales, tensor scale) of the formats'
    definitions, each scale step rounded to fp32 as they state."""
    x = x.double()
    if fmt in ("mxfp4", "mxfp8"):
        b = x.reshape(x.shape[0], -1, 32)
        a = b.abs().amax(2, keepdim=True)
        e = torch.frexp(a)[1] - 1 - (2 if fmt == "mxfp4" else 8)
        s = torch.where(a > 0, torch.ldexp(torch.ones_like(a), e.clamp(-127, 127)), torch.ones_like(a))
        d = _e2m1(b / s) if fmt == "mxfp4" else _e4m3(b / s)
        return (d * s).reshape(x.shape), 1.0
    amax = x.abs().max()
    if fmt == "fp8":
        s = _f32(amax / 448.0) if scale is None else scale.double()
        r = _f32(1.0 / s) if s > 0 else torch.zeros_like(s)
        return _e4m3(_f32(x * r)), s
    s = _f32(amax / 2688.0) if scale is None else scale.double()
    d = _f32(6.0 * s)
    b = x.reshape(x.shape[0], -1, 16)
    sb = _e4m3(_f32(b.abs().amax(2, keepdim=True) / d)) if d > 0 else torch.zeros_like(b[:, :, :1])
    S = _f32(sb * s)
    r = torch.where(S > 0, _f32(1.0 / S), torch.zeros_like(S))
    return (_e2m1(_f32(b * r)) * sb).reshape(x.shape), s


def _product(a, w, fmt, scale=None):
    """A W^T of the dequantized operands; A as bf16 (weight-only) or (decoded codes, scale)."""
    if isinstance(a, tuple):
        ad, s_a = a
    else:
        ad, s_a = (a.double(), 1.0) if fmt == "w4a16" else _quantized(a, fmt, scale)
    if w.shape[0] <= 16384:
        wd, s_w = _quantized(w, "nvfp4" if fmt == "w4a16" else fmt)
        return (ad @ wd.t()) * (s_a * s_w)
    s_w = _f32(w.abs().max().double() / 2688.0)  # a wide pool: one tensor scale, then in pieces
    return torch.cat([ad @ _quantized(p, "nvfp4", s_w.float())[0].t() for p in w.split(16384)], 1) * (s_a * s_w)


def exact(case, seed):
    x, w = _inputs(case, seed)
    if case["kind"] == "weights":
        d, s = _quantized(w["w"], case["fmt"])
        out = {"codes": None, "w": d * s}
        if case["fmt"] != "fp8":
            out["block_scales"] = None
        return out
    if case["kind"] == "fused":
        a = _quantized(x, "fp8")
        return {"y": _product(a, w["w"], "fp8"), "scale": a[1].reshape(1)}
    if case["kind"] == "linear":
        return {"y": _product(x, w["w"], case["fmt"], _static_scale(case) if case["static"] else None)}
    fmt, sc = case["fmt"], {s: _static_scale(case, s) for s in ("x", "v", "a", "u")}
    h = _f32(_product(x, w["qkv"], fmt, sc["x"])[:, 2 * HIDDEN:])
    a = _f32(_product(_quantized(h, fmt, sc["v"]), w["attn_out"], fmt))
    u = _product(_quantized(a, fmt, sc["a"]), w["mlp_up"], fmt)
    g = F.gelu(u.bfloat16(), approximate="tanh")
    return {"qkv_codes": None, "attn_out_codes": None, "mlp_up": u, "y": _product(g, w["mlp_down"], fmt, sc["u"])}


def tolerance(case):
    """About four times what was measured against exact() (2-norm, largest)."""
    if case["kind"] == "weights":
        return "exact"  # every step of the formats is one correctly rounded operation
    if case["kind"] == "block":
        # codes at a rounding boundary flip with the order of the sums and travel through the layers: FP8, whose matrix
        # instruction keeps about 16 bits of a sum, 0.1 % of the QKV codes, 0.6 % in mlp_up and 1.6 % in y; NVFP4,
        # whose products are exact, 3e-6 of the codes
        return {"rel": 0.03, "max": 0.6, "differ": 4e-3} if case["fmt"] == "fp8" else {"rel": 7e-3, "max": 0.1, "differ": 2e-5}
    if case["out"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}  # the rounding to bf16: 1.7e-3, 3.9e-3
    if case["kind"] == "fused" or case["fmt"] in ("fp8", "mxfp8"):
        return {"rel": 6e-5, "max": 7e-4}  # the FP8 matrix instruction's sums: 1.5e-5, 1.8e-4
    return {"rel": 1.2e-6, "max": 1.2e-5}  # fp32 sums of exact products: 3e-7, 2.8e-6
