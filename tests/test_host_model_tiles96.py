"""Staged tiles of 96 columns on the CPU execution model: the launches take them, and sampled workgroups of them compute the
oracle's product (tiles that start between two 64-row groups of scales, both scale layouts, two scale dwords of MXFP4)."""
import pytest

import test_host_model as fp8
import test_host_model_fp4 as fp4
from route_cases import launch
from test_host_model import MODES, hostmodel, run_case  # noqa: F401
from test_host_model_routes import routes

# format, M, N, K steps, BF16 output, padding of the rows of C (elements), tiled scales, bound on workgroups; kernel, tile
CASES = [
    (("fp8", 1000, 2880, 36, True, 0, True, 0), ("staged", 128, 96)),
    (("fp8", 897, 2785, 37, False, 3, False, 0), ("staged", 128, 96)),   # one row and one column in the last tiles
    (("fp4", 1000, 2850, 36, True, 0, True, 0), ("staged", 128, 96)),
    (("fp4", 900, 2880, 37, False, 0, False, 0), ("staged", 128, 96)),
    (("bf16", 900, 2817, 36, True, 0, False, 0), ("staged", 128, 96)),
    (("e5m2", 1000, 2880, 45, True, 0, False, 0), ("staged", 128, 96)),
    (("fp8", 200, 5120, 24, True, 0, True, 0), ("staged", 64, 96)),
    (("fp8", 193, 5089, 25, False, 1, False, 0), ("staged", 64, 96)),
    (("fp4", 200, 5120, 24, True, 0, False, 0), ("staged", 64, 96)),
    (("bf16", 200, 5100, 27, False, 0, False, 0), ("staged", 64, 96)),
]


def test_launches(hostmodel, tmp_path):  # noqa: F811
    calls = [c for c, _ in CASES]
    got = routes(hostmodel, tmp_path, [c[:5] + (c[2] + c[5],) + (0,) + c[6:] for c in calls])
    for (call, want), r in zip(CASES, got):
        assert r == launch(call, *want), call


@pytest.mark.parametrize("tiled", [True, False], ids=["tiled", "rowmajor"])
def test_sampled_workgroups(hostmodel, tmp_path, tiled):  # noqa: F811
    """Few units, so that small problems take these tiles; first, middle and last workgroup."""
    M, N = 230, 1500
    ops = fp8._operands(M, N, 24 * 128, seed=1)
    call = ("fp8", M, N, 24, False, N, 0, tiled, 0)
    assert routes(hostmodel, tmp_path, [call], WAVESIM_CUS=16)[0] == launch(call[:5] + (0, tiled, 0), "staged", 128, 96)
    line, out = fp8._gemm_case(tmp_path, M, N, 24 * 128, ops, False, N, tiled=tiled)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=16, WAVESIM_BLOCKS=4, **MODES[0])
    assert calls[0][0] == 0
    fp8._check_gemm(out, M, N, N, ops, False, expect_full=False)
    ops = fp4._fp4_operands(M, N, 24 * 256, seed=2)
    line, out = fp4._fp4_gemm_case(tmp_path, M, N, 24 * 256, ops, False, N, tag="4", tiled=tiled)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=16, WAVESIM_BLOCKS=4, **MODES[3])
    assert calls[0][0] == 0
    fp4._check_fp4_gemm(out, M, N, N, ops, False, expect_full=False)
