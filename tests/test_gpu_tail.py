"""Products whose 256x256 tiles overflow the units by a few: the rest is computed as quarters by a second launch. Each output
element goes through the same matrix instructions, so the bits are those of the product of half the rows."""
import os

import pytest
import torch

import paper_2506_08027_amd as mx
from route_cases import TAIL_SHAPES

pytestmark = [pytest.mark.gpu, pytest.mark.skipif("MXFP8_HOSTMODEL_LIB" in os.environ, reason="sizes for the hardware")]
LAYOUTS = {"tiled": mx.SCALES_TILED, "rowmajor": mx.SCALES_ROWMAJOR}


def _tensor(rows, cols, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((rows, cols), generator=g, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("shape", TAIL_SHAPES)
@pytest.mark.parametrize("layout", ["tiled", "rowmajor"])
@pytest.mark.parametrize("kind", ["bf16", "f32", "fp4", "simulated"])
def test_plain_products(shape, layout, kind):
    M, N, K = shape
    x, w = _tensor((M + 31) // 32 * 32, K, 1), _tensor((N + 31) // 32 * 32, K, 2)
    out = torch.float32 if kind == "f32" else torch.bfloat16
    lay = LAYOUTS[layout]

    def product(rows):
        if kind == "simulated":
            return mx.gemm_bf16(x[rows], w[:N], out)
        quantize, gemm = (mx.fp4_quantize, mx.fp4_gemm) if kind == "fp4" else (mx.quantize, mx.gemm)
        kk = 2 * K if kind == "fp4" else K   # 128-byte K steps of either format
        a, b = (quantize(torch.cat([t, t], 1) if kk > K else t, "rowwise", scale_layout=lay) for t in (x[rows.start // 32 * 32:(rows.stop + 31) // 32 * 32], w))
        m = rows.stop - rows.start
        cut = lambda q, s, r: (q[:r], s[:mx.mxfp8_scale_bytes(r, kk, lay)] if layout == "tiled" else s[:r])  # noqa: E731
        return gemm("fprop", *cut(a["q_row"], a["s_row"], m), *cut(b["q_row"], b["s_row"], N), out, lay)

    whole = product(slice(0, M))
    for rows in (slice(0, 2048), slice(2048, M)):
        part = product(rows)
        assert torch.equal(whole[rows].view(torch.int16 if out == torch.bfloat16 else torch.int32), part.view(torch.int16 if out == torch.bfloat16 else torch.int32))


@pytest.mark.parametrize("layout", ["tiled", "rowmajor"])
@pytest.mark.parametrize("ends", [[960, 960, 2752, 4352], [4352, 4352, 4352, 4352], [64, 2112, 2176, 4224]])
@pytest.mark.parametrize("k", [2048, 3584])
def test_grouped_products(layout, ends, k):
    """272 .. 304 tiles on 256 units; the last expert's rows may end before the operand does."""
    N, lay = 4096, LAYOUTS[layout]
    if layout == "rowmajor":
        ends = [max(0, e - 3) for e in ends]
    x = mx.quantize(_tensor(4352, k, 3), "rowwise", lay)
    ws = [mx.quantize(_tensor(N, k, 10 + e), "rowwise", lay) for e in range(4)]
    w_q = torch.stack([w["q_row"] for w in ws])
    w_s = torch.cat([w["s_row"] for w in ws]) if layout == "tiled" else torch.stack([w["s_row"] for w in ws])
    y = mx.gemm_grouped("fprop", x["q_row"], x["s_row"], w_q, w_s, torch.tensor(ends, dtype=torch.int32, device="cuda"), torch.bfloat16, lay)
    xr = mx.quantize(_tensor(4352, k, 3), "rowwise")
    begin = 0
    for e, end in enumerate(ends):
        if end > begin:
            wr = mx.quantize(_tensor(N, k, 10 + e), "rowwise")
            want = mx.gemm("fprop", xr["q_row"][begin:end], xr["s_row"][begin:end], wr["q_row"], wr["s_row"], torch.bfloat16)
            assert torch.equal(y[begin:end].view(torch.int16), want.view(torch.int16)), e
        begin = max(begin, end)
    assert torch.isnan(y[begin:]).all()   # filled by gemm_grouped; rows of no expert are not written
