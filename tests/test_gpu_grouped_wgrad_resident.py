"""Grouped weight gradients on resident workgroups (256x256 tiles, at least 128 of them, up to 128 experts): every output and scale
layout, whole and ragged tiles, loads from no step to most of them. Each expert's product must equal, bit for bit, the plain product
of its slice of the operands."""
import os

import pytest
import torch

import paper_2506_08027_amd as mx

pytestmark = [pytest.mark.gpu, pytest.mark.skipif("MXFP8_HOSTMODEL_LIB" in os.environ, reason="sizes for the hardware")]
LOADS = {
    "short": [1, 1, 0, 2, 0, 3, 1, 1, 1, 0, 0, 1, 2, 1, 1, 1] * 2,
    "one-heavy": [1] * 17 + [96] + [1, 0, 2, 1] * 4,           # its workgroups sit out rounds
    "two-heavy": [40, 3, 0, 2, 40, 3, 4, 1] + [2] * 24,
    "all-empty-but-one": [0] * 31 + [5],
    "128-experts": [2, 0, 1, 3] * 32,
    "129-experts": [2, 0, 1, 3] * 32 + [1],                    # one tile per workgroup
}


@pytest.mark.parametrize("load", list(LOADS))
@pytest.mark.parametrize("M,N", [(512, 768), (520, 776), (1024, 2048)])
@pytest.mark.parametrize("layout", [mx.SCALES_TILED, mx.SCALES_ROWMAJOR], ids=["tiled", "rowmajor"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_equals_the_plain_product_of_each_slice(load, M, N, layout, dtype):
    steps = LOADS[load]
    ends = [128 * sum(steps[:e + 1]) for e in range(len(steps))]
    K = ends[-1]
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    pad = lambda r: (r + 31) // 32 * 32  # noqa: E731
    src = [torch.randn((pad(r), K), generator=g, device="cuda").to(torch.bfloat16) for r in (M, N)]
    def operand(x, rows):
        q = mx.quantize(x.contiguous(), "rowwise", layout)
        return q["q_row"][:rows], q["s_row"][:mx.mxfp8_scale_bytes(rows, x.shape[1], layout)] if layout == mx.SCALES_TILED else q["s_row"][:rows]
    a, b = operand(src[0], M), operand(src[1], N)
    dw = mx.gemm_grouped("wgrad", *a, *b, torch.tensor(ends, dtype=torch.int32, device="cuda"), dtype, layout)
    bits, begin = torch.int32 if dtype == torch.float32 else torch.int16, 0
    for e, end in enumerate(ends):
        if end == begin:
            assert (dw[e] == 0).all(), e
        else:
            want = mx.gemm("wgrad", *operand(src[0][:, begin:end], M), *operand(src[1][:, begin:end], N), dtype, layout)
            assert torch.equal(dw[e].view(bits), want.view(bits)), e
        begin = end
