"""The resident product kernel on ragged problems (the last tiles are moved back to end with the operand) and with
256x192 tiles, on the CPU execution model of the kernels: both scale layouts (with tiled scales a moved tile begins
inside a 64-row group), several tiles per workgroup, all operand formats."""
import numpy as np
import pytest

import test_host_model as fp8
import test_host_model_fp4 as fp4
import test_host_model_simulated as sim
from test_host_model import MODES, hostmodel, run_case  # noqa: F401  (hostmodel is a fixture)

# M, N, K steps, BF16 output, tiled scales, compute units (ragged problems ignore the bound on workgroups), simulated workgroups, mode
CASES = [(2100, 4088, 3, True, True, 0, 3, 1), (2049, 4104, 2, True, False, 48, 2, 2), (2248, 3700, 3, False, True, 100, 2, 3)]


@pytest.mark.parametrize("case", CASES, ids=lambda s: "x".join(str(int(v)) for v in s))
def test_ragged_resident_gemm(hostmodel, tmp_path, case):
    M, N, steps, bf16, tiled, units, blocks, mode = case
    ops = fp8._operands(M, N, steps * 128, seed=M + N)
    line, out = fp8._gemm_case(tmp_path, M, N, steps * 128, ops, bf16, tiled=tiled, wg=2)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_BLOCKS=blocks, WAVESIM_CUS=units or 256, **MODES[mode])
    assert calls[0][0] == 0 and len(calls[0][1]) == blocks
    fp8._check_gemm(out, M, N, N, ops, bf16, expect_full=False)


def _tiles_of(workgroup, units, tiles_m, tiles_n):
    """(row, column) of the tiles that a resident workgroup walks over: XCD-contiguous ids, panels of 8 tile columns."""
    n, out = tiles_m * tiles_n, []
    for bid in range(workgroup, n, units):
        lid = (bid % 8) * (n // 8) + bid // 8 if bid < n // 8 * 8 else bid
        panel, rest = divmod(lid, 8 * tiles_m)
        width = min(8, tiles_n - panel * 8)
        out.append((rest // width, panel * 8 + rest % width))
    return out


# operand format, M, N, K steps, BF16 output: three by three 256x256 tiles, the last row and column of them moved back to a place
# inside a 64-row group of the tiled scales
HAND_OVERS = [("fp8", 760, 744, 5, True), ("fp8", 712, 744, 4, False), ("fp4", 760, 744, 4, True)]


@pytest.mark.parametrize("case", HAND_OVERS, ids=lambda s: "x".join(str(v) for v in s))
def test_ragged_resident_hand_over_between_tiles(hostmodel, tmp_path, case):
    """Two workgroups go from tiles in place to tiles moved back in M, in N and in both, and back: with tiled scales a lane's
    scale offset then differs from one tile to the next, for A and B separately, while both tiles' steps are in flight."""
    fmt, M, N, steps, bf16 = case
    moved = lambda t: (t[0] == 2, t[1] == 2)  # noqa: E731
    pairs = [(moved(a), moved(b)) for w in (0, 1) for a, b in zip(_tiles_of(w, 2, 3, 3)[:-1], _tiles_of(w, 2, 3, 3)[1:])]
    for axis in (0, 1):
        assert {(a[axis], b[axis]) for a, b in pairs} >= {(False, True), (False, False)}
    assert ((False, True), (False, False)) in pairs and (M - 256) % 64 and (N - 256) % 64
    mode = MODES[HAND_OVERS.index(case)]
    if fmt == "fp8":
        ops = fp8._operands(M, N, steps * 128, seed=M + N)
        line, out = fp8._gemm_case(tmp_path, M, N, steps * 128, ops, bf16, tiled=True)
    else:
        ops = fp4._fp4_operands(M, N, steps * 256, seed=M + N)
        line, out = fp4._fp4_gemm_case(tmp_path, M, N, steps * 256, ops, bf16, N, tiled=True)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=2, **mode)
    assert calls[0] == (0, [0, 1])   # two resident workgroups: everything is computed, the moved tiles among it
    (fp8._check_gemm if fmt == "fp8" else fp4._check_fp4_gemm)(out, M, N, N, ops, bf16)


def test_bounded_product_takes_256_tiles(hostmodel, tmp_path):
    """Whole 128x128 tiles on few workgroups: 256x256 tiles although there are few of them, the last ones moved back."""
    M, N, steps = 896, 512, 4
    ops = fp8._operands(M, N, steps * 128, seed=M + N)
    line, out = fp8._gemm_case(tmp_path, M, N, steps * 128, ops, True, tiled=True, wg=1)
    _, calls = run_case(hostmodel, tmp_path, [line], **MODES[2])
    assert calls[0] == (0, [0])
    fp8._check_gemm(out, M, N, N, ops, True)


def test_256x192_tiles(hostmodel, tmp_path):
    """[2048 x 6144]: 256 tiles of 256x192 where 256x256 tiles would leave a quarter of the units idle; and ragged."""
    for i, (M, N, steps, bf16, tiled) in enumerate(((2048, 6144, 9, True, True), (2040, 6136, 4, False, False))):
        ops = fp8._operands(M, N, steps * 128, seed=7 + i)
        line, out = fp8._gemm_case(tmp_path, M, N, steps * 128, ops, bf16, tiled=tiled, wg=128, tag=str(i))
        _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_BLOCKS=2, WAVESIM_CUS=128 if i else 256, **MODES[3 * i])
        assert calls[0] == (0, [0, 127])
        n = fp8._check_gemm(out, M, N, N, ops, bf16, expect_full=False)
        assert 3 * 256 * 192 < n <= 4 * 256 * 192


def test_256x192_tiles_other_operand_formats(hostmodel, tmp_path):
    M, N = 2048, 6144
    ops = fp4._fp4_operands(M, N, 1024, seed=3)
    line, out = fp4._fp4_gemm_case(tmp_path, M, N, 1024, ops, True, N, tiled=True)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_BLOCKS=2)
    assert calls[0][1] == [0, 255]
    fp4._check_fp4_gemm(out, M, N, N, ops, True, expect_full=False)
    ops = sim._operands(M, N, 320, seed=9)
    line, out = sim._case(tmp_path, M, N, 320, ops, True)
    _, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_BLOCKS=2, **MODES[3])
    assert calls[0][1] == [0, 255]
    sim._check(out, M, N, N, ops, True, expect_full=False)
