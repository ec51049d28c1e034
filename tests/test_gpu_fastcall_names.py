"""Passes and axes by name ("fprop", "both") take the binding's calls in C++ like the constants do."""
import os

import pytest
import torch

import paper_2506_08027_amd as mx
from paper_2506_08027_amd import binding

pytestmark = [pytest.mark.gpu, pytest.mark.skipif("MXFP8_HOSTMODEL_LIB" in os.environ, reason="the module takes tensors in GPU memory")]


def test_names_are_handled(monkeypatch):
    mx.load()
    codes, done = [], binding._done
    monkeypatch.setattr(binding, "_done", lambda rc, what: codes.append(rc) or done(rc, what))
    x = torch.ones((128, 256), dtype=torch.bfloat16, device="cuda")
    c = torch.empty((128, 128), dtype=torch.bfloat16, device="cuda")
    q = mx.quantize(x, "both")
    mx.mxfp8_quantize_ex(x, "both", **q)
    f4, f6 = mx.fp4_quantize(x, "rowwise"), mx.fp6_quantize(x, mx.E2M3, "rowwise")
    mx.mxfp8_fp4_quantize_ex(x, "rowwise", **f4)
    mx.mxfp8_fp6_quantize_ex(x, "rowwise", mx.E2M3, **f6)
    cq = mx.quantize(c, "both")
    codes.clear()
    mx.mxfp8_quantize_ex(x, "both", **q)
    mx.mxfp8_fp4_quantize_ex(x, "rowwise", **f4)
    mx.mxfp8_fp6_quantize_ex(x, "rowwise", mx.E2M3, **f6)
    mx.mxfp8_gemm_ex("fprop", q["q_row"], q["s_row"], q["q_row"], q["s_row"], c)
    mx.mxfp8_gemm_mode_ex("dgrad", q["q_row"], q["s_row"], mx.E5M2, q["q_row"], q["s_row"], mx.E4M3, c)
    mx.mxfp8_fp4_gemm_ex("fprop", f4["q_row"], f4["s_row"], f4["q_row"], f4["s_row"], c)
    mx.mxfp8_gemm_quantize_ex("fprop", q["q_row"], q["s_row"], q["q_row"], q["s_row"], c, "both", **{"c" + k: v for k, v in cq.items()})
    torch.cuda.synchronize()
    assert codes == [0] * 7
