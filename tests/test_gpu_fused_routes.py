"""mxfp8_gemm_quantize_ex on both sides of every line between one kernel and product-then-quantizer."""
import pytest
import torch

import paper_2506_08027_amd as mx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(128, 128, 512), (128, 128, 640), (256, 384, 256), (2048, 2048, 1024), (2048, 2048, 1152),
                                   (2816, 3072, 256), (4096, 4096, 256), (512, 1024, 384), (512, 1024, 512), (1024, 1536, 896), (1024, 1536, 1024),
                                   (1280, 2048, 1536), (1280, 2048, 1664), (1920, 2432, 896), (1920, 2432, 1024), (2560, 2560, 1536),
                                   (2560, 2560, 1664), (3328, 4096, 512), (4352, 4096, 512)])
@pytest.mark.parametrize("axis", ["rowwise", "colwise", "both"])
def test_fused_output_quantization_is_the_same_either_way(shape, axis):
    """Sizes on both sides of every line between one kernel and product-then-quantizer: the bytes are those of the two calls."""
    M, N, K = shape
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a, b = (mx.quantize(torch.randn((r, K), generator=g, device="cuda").to(torch.bfloat16), "rowwise", mx.SCALES_TILED) for r in (M, N))
    args = (a["q_row"], a["s_row"], b["q_row"], b["s_row"])
    out = mx.gemm_quantize("fprop", *args, axis=axis, scale_layout=mx.SCALES_TILED)
    c = mx.gemm("fprop", *args, torch.bfloat16, mx.SCALES_TILED)
    want = mx.quantize(c, axis, mx.SCALES_TILED)
    assert torch.equal(out["c"].view(torch.int16), c.view(torch.int16))
    for name, w in want.items():
        assert torch.equal(out[name], w), name
