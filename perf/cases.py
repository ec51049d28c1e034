"""The work that programs have this library do, as cases that can be timed and compared: whole linear-layer steps,
single products, the quantizers, and the extended paths (fused output quantization, mixture of experts, the simulated
BF16 path, MXFP4, MXFP6), from a few hundred tokens to the 8B-class shapes (hidden 4096, FFN 14336, 16384 tokens).

Every case calls the library's own entry points on buffers that the program keeps, as bench.py does. Tokens count the
rows of activations; h and o are the input and output widths of a linear layer; e experts. `layout` is the scale layout.
"""
import math

import torch

import paper_2506_08027_amd as mx

BLOCK = 32
LAYOUT = {"rowmajor": mx.SCALES_ROWMAJOR, "tiled": mx.SCALES_TILED}
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
ELEMENT = {"e4m3": mx.E4M3, "e5m2": mx.E5M2}
# element format: mantissa bits, exponent of the smallest normal, largest magnitude, exponent of the top binade, bits
FORMATS = {"e4m3": (3, -6, 448.0, 8, 8), "e5m2": (2, -14, 57344.0, 15, 8), "e2m1": (1, 0, 6.0, 2, 4), "e2m3": (3, 0, 7.5, 2, 6),
           "e3m2": (2, -2, 28.0, 4, 6)}


def listed():
    return [
        # The smallest training step that is run: a narrow layer on a short micro-batch, ten launches that each last a
        # few microseconds (quantize x, w, dy along both axes, three products, decode).
        {"name": "step_small", "op": "step", "tokens": 384, "h": 512, "o": 896, "grad": "bf16", "layout": "rowmajor"},
        # The benchmark's step: MLP up-projection of an 8B-class model at 8192 tokens, FP32 output gradient.
        {"name": "step_mlp_up", "op": "step", "tokens": 8192, "h": 4096, "o": 14336, "grad": "f32", "layout": "tiled"},
        # Forward product of the QKV layer for a few tokens (evaluating a trained model prompt by prompt).
        {"name": "fprop_few_tokens", "op": "gemm", "pass": "fprop", "m": 48, "n": 6144, "k": 4096, "a": "e4m3", "b": "e4m3",
         "out": "bf16", "layout": "rowmajor"},
        # Activation gradient of an unpadded batch: a token count and widths that no tile divides, 45 K steps.
        {"name": "dgrad_ragged", "op": "gemm", "pass": "dgrad", "m": 1000, "n": 2880, "k": 5760, "a": "e5m2", "b": "e4m3",
         "out": "bf16", "layout": "rowmajor"},
        # Forward product of the down-projection at 16384 tokens: the longest reduction and the largest product.
        {"name": "fprop_down_16384", "op": "gemm", "pass": "fprop", "m": 16384, "n": 4096, "k": 14336, "a": "e4m3", "b": "e4m3",
         "out": "bf16", "layout": "tiled"},
        # Quantizer on the benchmark's BF16 activations, both copies.
        {"name": "quantize_x", "op": "quantize", "rows": 8192, "cols": 4096, "src": "bf16", "axis": "both", "layout": "tiled"},
        # Quantizer on FP32 output gradients of an unpadded batch (rows that the 128-row tiles do not divide).
        {"name": "quantize_dy_ragged", "op": "quantize", "rows": 4128, "cols": 14336, "src": "f32", "axis": "both", "layout": "rowmajor"},
        # Forward product that hands the next layer its quantized input (both copies of the BF16 output).
        {"name": "fused_mlp_up", "op": "fused", "m": 4096, "n": 14336, "k": 4096, "axis": "both", "layout": "tiled"},
        # Mixture-of-experts layer, forward, activation gradient and weight gradient, unevenly loaded experts.
        {"name": "moe_step", "op": "moe", "tokens": 8192, "h": 2048, "o": 5632, "e": 8, "layout": "tiled"},
        # Simulated MX path: operands quantized, decoded to BF16, multiplied as BF16, FP32 result.
        {"name": "simulated_qkv", "op": "simulated", "tokens": 2048, "h": 4096, "o": 6144, "layout": "tiled"},
        # MXFP4 forward pass: activations quantized along both axes, product with the weight's row copy.
        {"name": "mxfp4_qkv", "op": "narrow", "tokens": 4096, "h": 4096, "o": 6144, "format": "e2m1", "axis": "both", "layout": "tiled"},
        # MXFP6 forward pass: activations quantized, product with a stored six-bit weight.
        {"name": "mxfp6_attn_out", "op": "narrow", "tokens": 4096, "h": 4096, "o": 4096, "format": "e2m3", "axis": "rowwise", "layout": "tiled"},
    ]


def _size(rng, lo, hi, of):
    """A multiple of `of` in [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / of)) * of))


def draw(rng):
    op = rng.choice(["step", "gemm", "gemm", "gemm", "quantize", "quantize", "fused", "moe", "simulated", "narrow", "narrow"])
    layout = rng.choice(["rowmajor", "tiled"])
    if op == "step":
        return {"op": op, "tokens": _size(rng, 256, 8192, 128), "h": _size(rng, 512, 4096, 128), "o": _size(rng, 512, 8192, 128),
                "grad": rng.choice(["bf16", "f32"]), "layout": layout}
    if op == "gemm":
        which = rng.choice(["fprop", "dgrad", "wgrad"])
        tokens = _size(rng, 16, 16384, 1) if which != "wgrad" else _size(rng, 256, 16384, 128)
        width = _size(rng, 512, 6144, 16)
        depth = _size(rng, 512, 8192, 128)
        m, n, k = (tokens, width, depth) if which != "wgrad" else (depth, width, tokens)
        return {"op": op, "pass": which, "m": m, "n": n, "k": k, "a": "e4m3" if which == "fprop" else rng.choice(["e4m3", "e5m2"]),
                "b": "e4m3", "out": "f32" if which == "wgrad" else "bf16", "layout": layout}
    if op == "quantize":
        return {"op": op, "rows": _size(rng, 64, 16384, 32), "cols": _size(rng, 512, 14336, 32), "src": rng.choice(["bf16", "f32"]),
                "axis": rng.choice(["rowwise", "colwise", "both", "both"]), "layout": layout}
    if op == "fused":
        big = rng.choice([True, False])  # the fused call takes whole tiles: of 256 where 128 of them fit, else of 128
        m, n = (_size(rng, 2816, 8192, 256), _size(rng, 3072, 8192, 256)) if big else (_size(rng, 256, 2048, 128), _size(rng, 512, 2048, 128))
        return {"op": op, "m": m, "n": n, "k": _size(rng, 512, 4096, 128), "axis": rng.choice(["rowwise", "both"]), "layout": layout}
    if op == "moe":
        return {"op": op, "tokens": _size(rng, 1024, 8192, 128), "h": _size(rng, 512, 2048, 128), "o": _size(rng, 512, 4096, 128),
                "e": rng.choice([4, 8, 16]), "layout": layout}
    if op == "simulated":
        return {"op": op, "tokens": _size(rng, 128, 4096, 32), "h": _size(rng, 512, 4096, 64), "o": _size(rng, 512, 4096, 32), "layout": layout}
    return {"op": op, "tokens": _size(rng, 128, 8192, 32), "h": _size(rng, 512, 4096, 256), "o": _size(rng, 512, 6144, 32),
            "format": rng.choice(["e2m1", "e2m1", "e2m3", "e3m2"]), "axis": rng.choice(["rowwise", "both"]), "layout": layout}


# ---- inputs ------------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _activations(g, rows, cols, dtype=torch.bfloat16):
    """N(0, 1) times a lognormal gain per channel, a few outlier channels 50 times larger."""
    gain = torch.exp(torch.randn(cols, generator=g, device="cuda"))
    gain[torch.randperm(cols, generator=g, device="cuda")[: max(1, cols // 1000)]] *= 50.0
    return (torch.randn((rows, cols), generator=g, device="cuda") * gain).to(dtype)


def _weights(g, rows, cols):
    return (0.02 * torch.randn((rows, cols), generator=g, device="cuda")).to(torch.bfloat16)


def _gradients(g, rows, cols, dtype):
    """N(0, 1e-3), 0.5 % of the entries 100 times larger."""
    x = 1e-3 * torch.randn((rows, cols), generator=g, device="cuda")
    x[torch.rand((rows, cols), generator=g, device="cuda") < 0.005] *= 100.0
    return x.to(dtype)


def _scales(rows, cols, layout):
    """A scale buffer; the places of a tiled one that belong to no block are zero."""
    n = mx.mxfp8_scale_bytes(rows, cols, LAYOUT[layout])
    return torch.zeros(n if layout == "tiled" else (rows, cols // BLOCK), dtype=torch.uint8, device="cuda")


def _copies(rows, cols, layout, axis="both", bits=8):
    """Buffers for the quantized copies of a [rows x cols] tensor."""
    out = {}
    if axis != "colwise":
        out["q_row"] = torch.empty((rows, cols * bits // 8), dtype=torch.uint8, device="cuda")
        out["s_row"] = _scales(rows, cols, layout)
    if axis != "rowwise":
        out["q_colT"] = torch.empty((cols, rows * bits // 8), dtype=torch.uint8, device="cuda")
        out["s_colT"] = _scales(cols, rows, layout)
    return out


def _operand_source(case, which):
    """How the operand `which` of a single product is drawn: rows, columns, kind of tensor."""
    rows = case["m"] if which == "a" else case["n"]
    kinds = {"fprop": {"a": "x", "b": "w"}, "dgrad": {"a": "dy", "b": "w"}, "wgrad": {"a": "dy", "b": "x"}}
    return rows, case["k"], kinds[case.get("pass", "fprop")][which]


def _source(g, rows, cols, kind):
    if kind == "x":
        return _activations(g, rows, cols)
    return _weights(g, rows, cols) if kind == "w" else _gradients(g, rows, cols, torch.bfloat16)


def _operand(src, element, layout):
    """Quantized row copy of src; a row count that the quantizer does not take is padded and the padding cut off."""
    rows, cols = src.shape
    padded = (rows + 31) // 32 * 32
    if padded != rows:
        src = torch.cat([src, torch.zeros((padded - rows, cols), dtype=src.dtype, device="cuda")])
    q = _copies(padded, cols, layout, "rowwise")
    mx.mxfp8_quantize_mode_ex(src, mx.ROWWISE, ELEMENT[element], mx.SCALE_ROUND_UP, q["q_row"], q["s_row"], scale_layout=LAYOUT[layout])
    s = q["s_row"][: mx.mxfp8_scale_bytes(rows, cols, LAYOUT[layout])] if layout == "tiled" else q["s_row"][:rows]
    return q["q_row"][:rows], s


def _ends(g, tokens, experts):
    """Row numbers at which the experts' tokens end: uneven loads, whole multiples of 128, one expert without tokens."""
    share = torch.rand(experts, generator=g, device="cuda") + 0.4
    share[int(torch.randint(experts, (1,), generator=g, device="cuda"))] = 0.0
    ends = (torch.cumsum(share, 0) / share.sum() * (tokens // 128)).round().to(torch.int32) * 128
    ends[-1] = tokens
    return ends


def _tensors(case, seed):
    """The unquantized tensors of a case, from the seed alone."""
    g, op = _generator(seed), case["op"]
    if op == "step":
        return {"x": _activations(g, case["tokens"], case["h"]), "w": _weights(g, case["o"], case["h"]),
                "dy": _gradients(g, case["tokens"], case["o"], DTYPE[case["grad"]])}
    if op in ("gemm", "fused"):
        return {which: _source(g, *_operand_source(case, which)) for which in ("a", "b")}
    if op == "quantize":
        return {"x": _activations(g, case["rows"], case["cols"]) if case["src"] == "bf16" else
                _gradients(g, case["rows"], case["cols"], torch.float32)}
    if op == "moe":
        return {"x": _activations(g, case["tokens"], case["h"]), "dy": _gradients(g, case["tokens"], case["o"], torch.bfloat16),
                "w": [_weights(g, case["o"], case["h"]) for _ in range(case["e"])], "ends": _ends(g, case["tokens"], case["e"])}
    return {"x": _activations(g, case["tokens"], case["h"]), "w": _weights(g, case["o"], case["h"])}  # simulated, narrow


def _narrow_quantize(src, axis, fmt, copies, layout):
    axis = {"rowwise": mx.ROWWISE, "both": mx.BOTH}[axis]
    if fmt == "e2m1":
        mx.mxfp8_fp4_quantize_ex(src, axis, **copies, scale_layout=layout)
    else:
        mx.mxfp8_fp6_quantize_ex(src, axis, mx.E2M3 if fmt == "e2m3" else mx.E3M2, **copies, scale_layout=layout)


def prepare(case, seed):
    t, op, layout = _tensors(case, seed), case["op"], case["layout"]
    s = {"op": op, "layout": LAYOUT[layout]}
    empty = lambda rows, cols, dtype: torch.empty((rows, cols), dtype=DTYPE[dtype], device="cuda")  # noqa: E731
    if op == "step":
        T, H, O = case["tokens"], case["h"], case["o"]
        s.update(t, xq=_copies(T, H, layout), wq=_copies(O, H, layout), dyq=_copies(T, O, layout), y=empty(T, O, "bf16"),
                 dx=empty(T, H, "bf16"), dw=empty(O, H, "f32"), xd=empty(T, H, "bf16"))
    elif op == "gemm":
        s["pass"] = case["pass"]
        for which in ("a", "b"):
            s[which + "_element"] = ELEMENT[case[which]]
            s[which + "_q"], s[which + "_s"] = _operand(t[which], case[which], layout)
        s["c"] = empty(case["m"], case["n"], case["out"])
    elif op == "quantize":
        s.update(x=t["x"], axis=case["axis"], copies=_copies(case["rows"], case["cols"], layout, case["axis"]))
    elif op == "fused":
        for which in ("a", "b"):
            s[which + "_q"], s[which + "_s"] = _operand(t[which], "e4m3", layout)
        s.update(axis=case["axis"], c=empty(case["m"], case["n"], "bf16"),
                 copies={"c" + k: v for k, v in _copies(case["m"], case["n"], layout, case["axis"]).items()})
    elif op == "moe":
        T, H, O, E = case["tokens"], case["h"], case["o"], case["e"]
        xq, dyq = mx.quantize(t["x"], "both", LAYOUT[layout]), mx.quantize(t["dy"], "both", LAYOUT[layout])
        wq = [mx.quantize(w, "both", LAYOUT[layout]) for w in t["w"]]
        s.update(x=xq, dy=dyq, ends=t["ends"], w={k: (torch.stack if k.startswith("q") else torch.cat)([w[k] for w in wq]) for k in wq[0]},
                 y=empty(T, O, "bf16"), dx=empty(T, H, "bf16"), dw=torch.empty((E, O, H), dtype=torch.float32, device="cuda"))
    elif op == "simulated":
        T, H, O = case["tokens"], case["h"], case["o"]
        s.update(t, xq=_copies(T, H, layout, "rowwise"), wq=_copies(O, H, layout, "rowwise"), x16=empty(T, H, "bf16"),
                 w16=empty(O, H, "bf16"), y=empty(T, O, "f32"))
    else:
        T, H, O, bits = case["tokens"], case["h"], case["o"], FORMATS[case["format"]][4]
        wq = _copies(O, H, layout, "rowwise", bits)
        _narrow_quantize(t["w"], "rowwise", case["format"], wq, LAYOUT[layout])
        s.update(x=t["x"], format=case["format"], axis=case["axis"], xq=_copies(T, H, layout, case["axis"], bits), wq=wq)
    return s


# ---- one pass ------------------------------------------------------------------------------------------------------

def run(s):
    op, lay = s["op"], s["layout"]
    if op == "step":
        xq, wq, dyq = s["xq"], s["wq"], s["dyq"]
        mx.mxfp8_quantize_ex(s["x"], mx.BOTH, **xq, scale_layout=lay)
        mx.mxfp8_quantize_ex(s["w"], mx.BOTH, **wq, scale_layout=lay)
        mx.mxfp8_gemm_ex(mx.FPROP, xq["q_row"], xq["s_row"], wq["q_row"], wq["s_row"], s["y"], lay)
        mx.mxfp8_quantize_ex(s["dy"], mx.BOTH, **dyq, scale_layout=lay)
        mx.mxfp8_gemm_ex(mx.DGRAD, dyq["q_row"], dyq["s_row"], wq["q_colT"], wq["s_colT"], s["dx"], lay)
        mx.mxfp8_gemm_ex(mx.WGRAD, dyq["q_colT"], dyq["s_colT"], xq["q_colT"], xq["s_colT"], s["dw"], lay)
        mx.mxfp8_dequantize_ex(xq["q_row"], xq["s_row"], s["xd"], lay)
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"], "xd": s["xd"], "xq": xq, "wq": wq, "dyq": dyq}
    if op == "gemm":
        if s["a_element"] == mx.E4M3 and s["b_element"] == mx.E4M3:
            mx.mxfp8_gemm_ex(s["pass"], s["a_q"], s["a_s"], s["b_q"], s["b_s"], s["c"], lay)
        else:
            mx.mxfp8_gemm_mode_ex(s["pass"], s["a_q"], s["a_s"], s["a_element"], s["b_q"], s["b_s"], s["b_element"], s["c"], lay)
        return {"c": s["c"]}
    if op == "quantize":
        mx.mxfp8_quantize_ex(s["x"], s["axis"], **s["copies"], scale_layout=lay)
        return s["copies"]
    if op == "fused":
        mx.mxfp8_gemm_quantize_ex(mx.FPROP, s["a_q"], s["a_s"], s["b_q"], s["b_s"], s["c"], s["axis"], **s["copies"], scale_layout=lay)
        return {"c": s["c"], **s["copies"]}
    if op == "moe":
        x, dy, w = s["x"], s["dy"], s["w"]
        mx.mxfp8_gemm_grouped_ex(mx.FPROP, x["q_row"], x["s_row"], w["q_row"], w["s_row"], s["ends"], s["y"], lay)
        mx.mxfp8_gemm_grouped_ex(mx.DGRAD, dy["q_row"], dy["s_row"], w["q_colT"], w["s_colT"], s["ends"], s["dx"], lay)
        mx.mxfp8_gemm_grouped_ex(mx.WGRAD, dy["q_colT"], dy["s_colT"], x["q_colT"], x["s_colT"], s["ends"], s["dw"], lay)
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    if op == "simulated":
        for name in ("x", "w"):
            q = s[name + "q"]
            mx.mxfp8_quantize_ex(s[name], mx.ROWWISE, **q, scale_layout=lay)
            mx.mxfp8_dequantize_ex(q["q_row"], q["s_row"], s[name + "16"], lay)
        mx.mxfp8_gemm_bf16(s["x16"], s["w16"], s["y"])
        return {"y": s["y"], "x16": s["x16"], "w16": s["w16"], "xq": s["xq"], "wq": s["wq"]}
    xq, wq = s["xq"], s["wq"]
    _narrow_quantize(s["x"], s["axis"], s["format"], xq, lay)
    if s["format"] == "e2m1":
        y = mx.fp4_gemm("fprop", xq["q_row"], xq["s_row"], wq["q_row"], wq["s_row"], torch.bfloat16, lay)
    else:
        el = mx.E2M3 if s["format"] == "e2m3" else mx.E3M2
        y = mx.fp6_gemm("fprop", xq["q_row"], xq["s_row"], el, wq["q_row"], wq["s_row"], el, torch.bfloat16, lay)
    return {"y": y, "xq": xq}


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    op = case["op"]
    copy = lambda bits: bits / 8 + 1 / BLOCK  # noqa: E731  bytes per element of one quantized copy
    if op == "quantize":
        n = case["rows"] * case["cols"]
        return {"bytes": n * ((2 if case["src"] == "bf16" else 4) + copy(8) * (2 if case["axis"] == "both" else 1)), "flops": 0}
    if op == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": (m + n) * k * copy(8) + m * n * (2 if case["out"] == "bf16" else 4), "flops": 2 * m * n * k}
    if op == "fused":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": (m + n) * k * copy(8) + m * n * (2 + copy(8) * (2 if case["axis"] == "both" else 1)), "flops": 2 * m * n * k}
    T, H, O = case["tokens"], case["h"], case["o"]
    if op == "step":  # every tensor read and every copy and result written once
        g = 4 if case["grad"] == "f32" else 2
        return {"bytes": (T * H + O * H) * (2 + 2 * copy(8)) + T * O * (g + 2 * copy(8)) + T * O * 2 + T * H * 2 + O * H * 4 + T * H * 2,
                "flops": 6 * T * H * O}
    if op == "moe":
        return {"bytes": 2 * (T * H + T * O + case["e"] * O * H) * copy(8) + T * O * 2 + T * H * 2 + case["e"] * O * H * 4,
                "flops": 6 * T * H * O}
    if op == "simulated":
        return {"bytes": (T * H + O * H) * (2 + copy(8) + 2) + T * O * 4, "flops": 2 * T * H * O}
    bits = FORMATS[case["format"]][4]
    return {"bytes": T * H * (2 + copy(bits) * (2 if case["axis"] == "both" else 1)) + O * H * copy(bits) + T * O * 2, "flops": 2 * T * H * O}


def tolerance(case):
    """Measured against exact(): products of MXFP8 operands are 4e-5 .. 8e-5 off in the 2-norm (the matrix instruction
    cuts products short inside groups of eight), plus 1.7e-3 where the result is stored as BF16; the BF16 products of
    the simulated path are 1.5e-7 off. About four times that is stated. Quantized bytes of the inputs do not differ;
    those of a fused product's output may where its last bit does."""
    op = case["op"]
    if op == "quantize":
        return "exact"
    if op == "simulated":
        return {"rel": 1e-5}
    if op == "gemm":
        return {"rel": 3e-4 if case["out"] == "f32" else 7e-3}
    if op == "fused":
        return {"rel": 7e-3, "differ": 1e-3}
    return {"rel": 7e-3}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------

def _rounded(x, fmt):
    """The values that x [rows x cols] has after quantization along its rows, in float64: blocks of 32, the scale the
    smallest power of two (from 2^-127) with amax <= largest * scale, elements rounded to nearest, ties to even."""
    mant, emin, largest, top, _ = FORMATS[fmt]
    v = x.to(torch.float64).reshape(x.shape[0], -1, BLOCK)
    amax = v.abs().amax(-1, keepdim=True)
    frac, exp = torch.frexp(amax)                     # amax = frac * 2^exp, frac in [0.5, 1)
    n = exp.to(torch.float64) - 1 - top + (frac * 2 > largest / 2.0 ** top).to(torch.float64)
    scale = torch.exp2(torch.where(amax > 0, n, torch.full_like(n, -127.0)).clamp(-127, 127))
    t = v / scale
    e = (torch.frexp(t.abs())[1].to(torch.float64) - 1).clamp(emin, top)
    step = torch.exp2(e - mant)
    return ((t / step).round() * step).clamp(-largest, largest).mul(scale).reshape(x.shape)


def _product(a, b):
    return a @ b.t()


def exact(case, seed):
    t, op = _tensors(case, seed), case["op"]
    if op == "quantize":
        return None
    if op == "step":
        r = lambda v: _rounded(v, "e4m3")  # noqa: E731
        x, w, dy = t["x"], t["w"], t["dy"]
        none = {"q_row": None, "s_row": None, "q_colT": None, "s_colT": None}
        return {"y": _product(r(x), r(w)), "dx": _product(r(dy), r(w.t())), "dw": _product(r(dy.t()), r(x.t())), "xd": r(x),
                "xq": none, "wq": none, "dyq": none}
    if op == "gemm":
        return {"c": _product(_rounded(t["a"], case["a"]), _rounded(t["b"], case["b"]))}
    if op == "fused":
        return {"c": _product(_rounded(t["a"], "e4m3"), _rounded(t["b"], "e4m3"))}
    if op == "moe":
        r = lambda v: _rounded(v, "e4m3")  # noqa: E731
        T, H, O, E = case["tokens"], case["h"], case["o"], case["e"]
        f64 = dict(dtype=torch.float64, device="cuda")
        y, dx, dw = torch.zeros((T, O), **f64), torch.zeros((T, H), **f64), torch.zeros((E, O, H), **f64)
        x, dy, x_t, dy_t = r(t["x"]), r(t["dy"]), r(t["x"].t()), r(t["dy"].t())
        begin = 0
        for e, end in enumerate(t["ends"].tolist()):
            if end > begin:
                y[begin:end] = _product(x[begin:end], r(t["w"][e]))
                dx[begin:end] = _product(dy[begin:end], r(t["w"][e].t()))
                dw[e] = _product(dy_t[:, begin:end], x_t[:, begin:end])
            begin = end
        return {"y": y, "dx": dx, "dw": dw}
    if op == "simulated":
        x, w = _rounded(t["x"], "e4m3"), _rounded(t["w"], "e4m3")
        return {"y": _product(x, w), "x16": x, "w16": w}
    return {"y": _product(_rounded(t["x"], case["format"]), _rounded(t["w"], case["format"]))}
