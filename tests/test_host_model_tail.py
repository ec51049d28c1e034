"""The quarters of 256x256 tiles that a second launch computes where the tiles do not fill the last round over the units, on the
CPU execution model (devices of a few units, first and last workgroup of each launch)."""
import numpy as np
import pytest

from test_host_model import _check_gemm, _gemm_case, _operands as _plain_operands, hostmodel, run_case  # noqa: F401
from test_host_model_grouped import _case, _check, _operands

pytestmark = pytest.mark.slow


@pytest.mark.parametrize("bf16,tiled", [(True, True), (False, False)], ids=["bf16-tiled", "f32-rowmajor"])
def test_plain_product(hostmodel, tmp_path, bf16, tiled):  # noqa: F811
    """Nine ragged tiles on eight units: the ninth as four quarters, the last of them 60 x 120."""
    M, N, K = 700, 760, 28 * 128
    ops = _plain_operands(M, N, K, seed=700)
    line, out = _gemm_case(tmp_path, M, N, K, ops, bf16=bf16, tiled=tiled, ldc=N + 8)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=8, WAVESIM_BLOCKS=2)
    assert calls[0][0] == 0
    written = _check_gemm(out, M, N, N + 8, ops, bf16, expect_full=False)
    assert written > 128 * 128 + 60 * 120   # tiles of the first launch, first and last quarter


@pytest.mark.parametrize("tiled", [True, False])
def test_grouped_product(hostmodel, tmp_path, tiled):  # noqa: F811
    """128 tiles of three experts on 120 units: the last eight as quarters, rows behind an expert's end left alone."""
    M, N, K = 2048, 4096, 16 * 128
    ends = [448, 1024, 2048] if tiled else [400, 1003, 2001]
    ops = _operands(M, N, K, len(ends), seed=61)
    line, out = _case(tmp_path, M, N, K, ops, ends, bf16=True, tiled=tiled)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=120, WAVESIM_BLOCKS=2)
    assert calls[0][0] == 0
    assert _check(out, M, N, N, ops, ends, True, expect_full=False) > 2 * 200 * 256
