"""The staged product kernel (problems of at least four K steps that 256x256 tiles cannot spread over the chip) on the
CPU execution model of the kernels: ring wrap-around, steps that are not a multiple of the ring or of the four-step
scale requests, tiles that end inside a row group, one-row and one-column remainders, several tiles per workgroup."""
import numpy as np
import pytest

import test_host_model as fp8
import test_host_model_fp4 as fp4
import test_host_model_gemm_modes as modes
import test_host_model_simulated as sim
from route_cases import launch
from test_host_model import MODES, hostmodel, run_case  # noqa: F401  (hostmodel is a fixture)
from test_host_model_routes import routes

# M, N, K steps, BF16 output, leading dimension - N, tiled scales, workgroup bound
SHAPES = [(1, 16, 4, False, 0, False, 0), (65, 129, 5, True, 7, True, 0), (200, 136, 8, True, 0, False, 0),
          (130, 72, 9, False, 4, False, 0), (192, 80, 12, True, 8, True, 0), (33, 255, 7, False, 1, True, 0),
          (384, 256, 12, True, 0, False, 2), (384, 384, 11, False, 4, True, 3)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(int(v)) for v in s))
def test_staged_gemm_edges(hostmodel, tmp_path, shape):
    M, N, steps, bf16, pad, tiled, wg = shape
    ops = fp8._operands(M, N, steps * 128, seed=M + N)
    if wg:   # several 128x128 tiles per workgroup (with fewer K steps they would go to the resident kernel)
        call = ("fp8", M, N, steps, bf16, pad, tiled, wg)
        assert routes(hostmodel, tmp_path, [call[:5] + (N + pad, 0, tiled, wg)])[0] == launch(call, "staged", 128, 128)
    line, out = fp8._gemm_case(tmp_path, M, N, steps * 128, ops, bf16, N + pad, tiled=tiled, wg=wg)
    for mode in (MODES[0], MODES[3]):
        _, calls = run_case(hostmodel, tmp_path, [line], **mode)
        assert calls[0][0] == 0 and (not wg or calls[0][1] == list(range(wg)))
        fp8._check_gemm(out, M, N, N + pad, ops, bf16)


def test_staged_gemm_128_tiles_sampled_workgroups(hostmodel, tmp_path):
    """128x128 tiles (at least 128 of them), ragged in both directions, both forms of row-major scale requests."""
    for i, steps in enumerate((8, 6)):
        M, N = 1400 + i, 1500 + 4 * i
        ops = fp8._operands(M, N, steps * 128, seed=5 + i)
        line, out = fp8._gemm_case(tmp_path, M, N, steps * 128, ops, True, N, tag=str(i))
        _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_BLOCKS=3, **MODES[3 * i])
        assert calls[0][0] == 0
        fp8._check_gemm(out, M, N, N, ops, True, expect_full=False)


def test_staged_gemm_other_operand_formats(hostmodel, tmp_path):
    """MXFP4 (two scale dwords per row and step), BF16 (no scales) and E5M2 operands."""
    for i, (tiled, bf16) in enumerate(((True, True), (False, False))):
        M, N, K = 70 + i, 200 - 8 * i, 1024 + 256 * i
        ops = fp4._fp4_operands(M, N, K, seed=3 + i)
        line, out = fp4._fp4_gemm_case(tmp_path, M, N, K, ops, bf16, N, tag=f"f{i}", tiled=tiled)
        _, calls = run_case(hostmodel, tmp_path, [line], **MODES[3 * i])
        assert calls[0][0] == 0
        fp4._check_fp4_gemm(out, M, N, N, ops, bf16)
    M, N, K = 90, 136, 320
    ops = sim._operands(M, N, K, seed=9)
    line, out = sim._case(tmp_path, M, N, K, ops, False)
    _, calls = run_case(hostmodel, tmp_path, [line])
    assert calls[0][0] == 0
    sim._check(out, M, N, N, ops, False)
    M, N, K = 100, 64, 640
    ops = modes._operands(M, N, K, 1, 0, seed=11)
    val, written = modes._run(hostmodel, tmp_path, M, N, K, 1, 0, ops)
    ref, absum = modes.oracle.gemm_mode(ops[0], ops[1], "e5m2", ops[2], ops[3], "e4m3")
    assert written.all() and (np.abs(val - ref) <= K // 128 * 2.0 ** -24 * absum + 1e-300).all()
