"""The binding's calls in C++ against the same calls through Python's checks: the same results for every form that both take, the
same refusals for what is refused."""
import os

import pytest
import torch

import paper_2506_08027_amd as mx
from paper_2506_08027_amd import binding

pytestmark = [pytest.mark.gpu, pytest.mark.skipif("MXFP8_HOSTMODEL_LIB" in os.environ, reason="the module takes tensors in GPU memory")]
TILED, ROWMAJOR = mx.SCALES_TILED, mx.SCALES_ROWMAJOR


@pytest.fixture(autouse=True)
def module_is_there():
    mx.load()
    assert binding._fast is not None, "paper_2506_08027_amd/_fastcall.so is not built"


def _u8(*shape):
    return torch.zeros(shape, dtype=torch.uint8, device="cuda")


def _x(rows, cols, dtype=torch.bfloat16, ld=None):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    return torch.randn((rows, ld or cols), generator=g, device="cuda").to(dtype)[:, :cols]


def _scale(rows, cols, layout):
    return _u8(mx.mxfp8_scale_bytes(rows, cols, layout)) if layout == TILED else _u8(rows, cols // 32)


def _copies(rows, cols, layout, num=1, den=1):
    return dict(q_row=_u8(rows, cols * num // den), s_row=_scale(rows, cols, layout), q_colT=_u8(cols, rows * num // den), s_colT=_scale(cols, rows, layout))


def _both_ways(call, outputs):
    """call() with and without the module; the outputs' bytes after each."""
    got = []
    for fast in (binding._fast, None):
        for o in outputs:
            o.view(torch.uint8).fill_(0x5A) if o.is_contiguous() else o.fill_(1)
        keep, binding._fast = binding._fast, fast
        try:
            call()
        finally:
            binding._fast = keep
        torch.cuda.synchronize()
        got.append([o.clone() for o in outputs])
    for a, b in zip(*got):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


@pytest.mark.parametrize("layout", [TILED, ROWMAJOR])
@pytest.mark.parametrize("dtype,ld", [(torch.bfloat16, None), (torch.float32, None), (torch.bfloat16, 168), (torch.float32, 164)])
def test_quantizers(layout, dtype, ld):
    x = _x(96, 160, dtype, ld)
    for axis in (mx.ROWWISE, mx.COLWISE, mx.BOTH, "rowwise"):
        c = _copies(96, 160, layout)
        _both_ways(lambda: mx.mxfp8_quantize_ex(x, axis, **c, scale_layout=layout), list(c.values()))  # noqa: B023
        _both_ways(lambda: mx.mxfp8_quantize_mode_ex(x, axis, mx.E5M2, mx.SCALE_OCP_V1, **c, scale_layout=layout), list(c.values()))  # noqa: B023
    c4, c6 = _copies(96, 160, layout, 1, 2), _copies(96, 160, layout, 3, 4)
    _both_ways(lambda: mx.mxfp8_fp4_quantize_ex(x, mx.BOTH, **c4, scale_layout=layout), list(c4.values()))
    _both_ways(lambda: mx.mxfp8_fp6_quantize_ex(x, mx.BOTH, mx.E3M2, **c6, scale_layout=layout), list(c6.values()))
    row = {k: v for k, v in _copies(96, 160, layout).items() if k.endswith("row")}
    _both_ways(lambda: mx.mxfp8_quantize_ex(x, mx.ROWWISE, **row, scale_layout=layout), list(row.values()))


@pytest.mark.parametrize("layout", [TILED, ROWMAJOR])
@pytest.mark.parametrize("out,ldc", [(torch.bfloat16, None), (torch.float32, None), (torch.float32, 101)])
def test_products_and_decode(layout, out, ldc):
    M, N, K = 70, 96, 256
    a, b = mx.quantize(_x(96, K), "both", layout), mx.quantize(_x(N, K), "both", layout)
    a_q, a_s = a["q_row"][:M], a["s_row"] if layout == TILED else a["s_row"][:M]
    args = (a_q, a_s, b["q_row"], b["s_row"])
    c = torch.zeros((M, ldc or N), dtype=out, device="cuda")[:, :N]
    for which in (mx.FPROP, "wgrad"):
        _both_ways(lambda: mx.mxfp8_gemm_ex(which, *args, c, layout), [c])  # noqa: B023
    _both_ways(lambda: mx.mxfp8_gemm_mode_ex(mx.DGRAD, a_q, a_s, mx.E5M2, b["q_row"], b["s_row"], mx.E4M3, c, layout, 3), [c])
    x, w = _x(M, K), _x(N, K)
    _both_ways(lambda: mx.mxfp8_gemm_bf16(x, w, c), [c])
    f = [mx.fp4_quantize(_x(r, K), "rowwise", layout) for r in (96, N)]
    c4 = torch.zeros((96, N), dtype=out, device="cuda")
    _both_ways(lambda: mx.mxfp8_fp4_gemm_ex(mx.FPROP, f[0]["q_row"], f[0]["s_row"], f[1]["q_row"], f[1]["s_row"], c4, layout), [c4])
    d = torch.zeros((96, ldc or K), dtype=out, device="cuda")[:, :K] if ldc is None or ldc >= K else torch.zeros((96, K + 12), dtype=out, device="cuda")[:, :K]
    _both_ways(lambda: mx.mxfp8_dequantize_ex(a["q_row"], a["s_row"], d, layout), [d])
    q = mx.quantize(_x(128, K), "both", layout)
    y, cq = torch.zeros((128, 128), dtype=torch.bfloat16, device="cuda"), {"c" + k: v for k, v in _copies(128, 128, layout).items()}
    _both_ways(lambda: mx.mxfp8_gemm_quantize_ex(mx.FPROP, q["q_row"], q["s_row"], q["q_row"], q["s_row"], y, mx.BOTH, **cq, scale_layout=layout), [y, *cq.values()])


def test_refusals_are_the_same():
    x, c = _x(64, 128), _copies(64, 128, ROWMAJOR)
    q = mx.quantize(x, "both")
    y = torch.zeros((64, 64), dtype=torch.bfloat16, device="cuda")
    gemm = lambda *a, **k: (lambda: mx.mxfp8_gemm_ex(mx.FPROP, *a, **k))  # noqa: E731
    ops = (q["q_row"], q["s_row"], q["q_row"], q["s_row"])
    calls = [
        lambda: mx.mxfp8_quantize_ex(x.cpu(), mx.BOTH, **c), lambda: mx.mxfp8_quantize_ex(x.half(), mx.BOTH, **c),
        lambda: mx.mxfp8_quantize_ex(x.t(), mx.BOTH, **c), lambda: mx.mxfp8_quantize_ex(x[:40], mx.BOTH, **c),
        lambda: mx.mxfp8_quantize_ex(x, 7, **c), lambda: mx.mxfp8_quantize_ex(x, mx.BOTH, q_row=c["q_row"], s_row=c["s_row"]),
        lambda: mx.mxfp8_quantize_ex(x, mx.BOTH, **c, scale_layout=5), lambda: mx.mxfp8_quantize_ex(x[:, 1:97], mx.ROWWISE, **c),
        lambda: mx.mxfp8_quantize_ex(x, mx.BOTH, **c, scale_layout=TILED), lambda: mx.mxfp8_fp4_quantize_ex(x, mx.BOTH, **c),
        lambda: mx.mxfp8_fp6_quantize_ex(x, mx.BOTH, 9, **_copies(64, 128, ROWMAJOR, 3, 4)),
        gemm(*ops, y.half()), gemm(*ops, y[:32]), gemm(*ops, y.t()[:, :64].t()), gemm(ops[0][:, :64], *ops[1:], y), gemm(ops[0].cpu(), *ops[1:], y),
        gemm(ops[0], ops[1][:, :2], *ops[2:], y), gemm(ops[0].t(), *ops[1:], y), gemm(*ops, y, max_workgroups=-1), gemm(*ops, y, 9),
        gemm(ops[0].view(torch.int8), *ops[1:], y), lambda: mx.mxfp8_gemm_ex("other", *ops, y), lambda: mx.mxfp8_gemm_ex(5, *ops, y),
        lambda: mx.mxfp8_dequantize_ex(q["q_row"], q["s_row"], y), lambda: mx.mxfp8_dequantize_ex(q["q_row"], q["s_row"], x.half()),
        lambda: mx.mxfp8_gemm_bf16(x, x.float(), y), lambda: mx.mxfp8_gemm_quantize_ex(mx.FPROP, *ops, y, mx.BOTH),
        lambda: mx.mxfp8_gemm_ex(mx.FPROP, *ops, None), lambda: mx.mxfp8_quantize_ex(None, mx.BOTH, **c),
    ]
    fast = binding._fast
    for i, call in enumerate(calls):
        seen = []
        for way in (fast, None):
            binding._fast = way
            try:
                call()
                seen.append(None)
            except Exception as e:  # noqa: BLE001
                seen.append((type(e), str(e)))
            finally:
                binding._fast = fast
        assert seen[0] == seen[1], (i, seen)
    torch.cuda.synchronize()
