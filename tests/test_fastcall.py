"""The binding's calls in C++ (csrc/fastcall.cpp) leave everything that is not the ordinary call to the binding's own checks."""
import importlib

import pytest
import torch


def test_other_arguments_are_not_handled():
    try:
        fast = importlib.import_module("paper_2506_08027_amd._fastcall")
    except ImportError:
        pytest.skip("not built")
    q, s, x = torch.zeros((32, 128), dtype=torch.uint8), torch.zeros((32, 4), dtype=torch.uint8), torch.zeros((32, 128))
    for args in ((), (1, 2, 3), (x, 3, 0, 0, q, s, None, None, 0, 0), ("src",) * 10, (None,) * 10, (2 ** 80,) * 10):
        for call in (fast.quantize, fast.gemm, fast.gemm_mode, fast.dequantize, fast.gemm_bf16, fast.gemm_quantize, fast.fp4_quantize, fast.fp4_gemm,
                     fast.fp6_quantize):
            assert call(*args) == -1
    assert fast.gemm(0, q, s, q, s, x, 0, 0, 0) == -1   # tensors in host memory
    with pytest.raises(TypeError):
        fast.bind(3)
