"""What the binding says first about a call with several mistakes: the tensors are looked at before the stream is asked for, on a
machine without a GPU too, with and without the calls in C++."""
import os
import sys

import pytest
import torch

import paper_2506_08027_amd as mx
from paper_2506_08027_amd import binding

pytestmark = pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="the library is not built")


def _calls(stream, which):
    """Every call that csrc/fastcall.cpp knows, on host tensors. which: the pass or axis."""
    q, s, x = torch.zeros((128, 256), dtype=torch.uint8), torch.zeros((128, 8), dtype=torch.uint8), torch.zeros((128, 256))
    c = torch.zeros((128, 128))
    return [
        lambda: mx.mxfp8_quantize_ex(x, which, q, s, stream=stream), lambda: mx.mxfp8_quantize_mode_ex(x, which, mx.E5M2, 0, q, s, stream=stream),
        lambda: mx.mxfp8_gemm_ex(which, q, s, q, s, c, stream=stream), lambda: mx.mxfp8_gemm_mode_ex(which, q, s, mx.E4M3, q, s, mx.E4M3, c, stream=stream),
        lambda: mx.mxfp8_gemm_bf16(x, x, c, stream=stream), lambda: mx.mxfp8_gemm_quantize_ex(which, q, s, q, s, c, which, stream=stream),
        lambda: mx.mxfp8_dequantize_ex(q, s, x, stream=stream), lambda: mx.mxfp8_fp4_quantize_ex(x, which, q, s, stream=stream),
        lambda: mx.mxfp8_fp4_gemm_ex(which, q, s, q, s, c, stream=stream), lambda: mx.mxfp8_fp6_quantize_ex(x, which, mx.E2M3, q, s, stream=stream),
    ]


@pytest.mark.parametrize("fast", [True, False], ids=["module", "python"])
@pytest.mark.parametrize("stream", [None, "no stream"])
@pytest.mark.parametrize("which", [1, "both", ["not", "hashable"]])
def test_host_tensors_are_reported_before_the_stream(monkeypatch, fast, stream, which):
    mx.load()
    if not fast:
        monkeypatch.setattr(binding, "_fast", None)
    elif binding._fast is None:
        pytest.skip("the calls in C++ are not built")
    for call in _calls(stream, which):
        with pytest.raises(ValueError, match="all tensors must live in GPU memory"):
            call()


def test_calls_in_cpp_that_cannot_be_loaded_are_reported(monkeypatch):
    lib = mx.load()
    monkeypatch.setitem(sys.modules, "paper_2506_08027_amd._fastcall", None)   # what an import of it then raises
    monkeypatch.delattr(sys.modules["paper_2506_08027_amd"], "_fastcall", raising=False)
    with pytest.warns(RuntimeWarning, match="cannot be loaded"):
        assert binding._bind_fastcall(lib) is None
