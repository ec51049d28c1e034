"""The quarters of 256x256 tiles that are computed where the tiles do not fill the last round over the units, on the CPU execution
model (devices of a few units): by a second launch of a plain product, at the end of the same launch by a grouped one."""
import numpy as np
import pytest

from route_cases import launch
from test_host_model import _check_gemm, _gemm_case, _operands as _plain_operands, hostmodel, run_case  # noqa: F401
from test_host_model_grouped import _case, _check, _operands


def _launches(res):
    """[(workgroups, LDS bytes)] of the launches of the only call."""
    line, = [v for v in res.stdout.splitlines() if v.startswith("launches")]
    return [tuple(int(x) for x in v.split(":")) for v in line.split()[1:]]


def _written(out, M, ldc, N, bf16):
    """Where C was written."""
    raw = np.full(M * ldc, 0xA5A5 if bf16 else 0xA5A5A5A5, np.uint16 if bf16 else np.uint32)
    raw[:(M - 1) * ldc + N] = np.fromfile(out, raw.dtype)
    return raw.reshape(M, ldc)[:, :N] != (0xA5A5 if bf16 else 0xA5A5A5A5)


def _area(M, N, *blocks):
    mask = np.zeros((M, N), bool)
    for rows, cols in blocks:
        mask[rows, cols] = True
    return mask


@pytest.mark.parametrize("which,bf16,tiled", [(1, True, True), pytest.param(1, False, False, marks=pytest.mark.slow),
                                              pytest.param(0, True, True, marks=pytest.mark.slow)], ids=["quarters-bf16-tiled", "quarters-f32-rowmajor", "tiles"])
def test_plain_product(hostmodel, tmp_path, which, bf16, tiled):  # noqa: F811
    """Nine ragged tiles on eight units: eight in the first launch, the ninth (188 rows, 248 columns) as four quarters in the second."""
    M, N, K = 700, 760, 28 * 128
    ops = _plain_operands(M, N, K, seed=700)
    line, out = _gemm_case(tmp_path, M, N, K, ops, bf16=bf16, tiled=tiled, ldc=N + 8)
    res, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=8, WAVESIM_ONLY=which, **({} if which else {"WAVESIM_BLOCKS": 2}))
    assert calls[0][0] == 0
    call = ("fp8", M, N, 28, bf16, 8, tiled, 0)
    assert _launches(res) == [(8, launch(call, "resident", 256, 256)[1]), (4, launch(call, "staged", 128, 128)[1])]
    _check_gemm(out, M, N, N + 8, ops, bf16, expect_full=False)
    written, ninth = _written(out, M, N + 8, N, bf16), _area(M, N, (slice(512, M), slice(512, N)))
    if which:
        assert np.array_equal(written, ninth)
    else:
        assert written.sum() >= 2 * 188 * 248 and not (written & ninth).any()


@pytest.mark.parametrize("tiled,blocks,wg", [(True, 1, 0), pytest.param(False, 3, 0, marks=pytest.mark.slow),
                                             pytest.param(True, 3, 128, marks=pytest.mark.slow)])
def test_grouped_product(hostmodel, tmp_path, tiled, blocks, wg):  # noqa: F811
    """144 tiles of three experts on 128 units, in one launch: the workgroups go on with the quarters of the last sixteen, which
    are four columns of the last expert's tiles; rows behind an expert's end are left alone. First, middle and last workgroup. A
    bound of as many workgroups as there are units is none."""
    M, N, K = 2048, 4096, 16 * 128
    ends = [448, 1024, 2048] if tiled else [400, 1003, 2001]
    ops = _operands(M, N, K, len(ends), seed=61)
    line, out = _case(tmp_path, M, N, K, ops, ends, bf16=True, tiled=tiled, wg=wg)
    res, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=128, WAVESIM_BLOCKS=blocks)
    assert calls[0] == (0, [0, 63, 127][:blocks])
    assert _launches(res) == [(128, launch(("fp8", M, N, 16, True, 0, tiled, 0), "resident", 256, 256)[1])]
    _check(out, M, N, N, ops, ends, True, expect_full=False)
    written = _written(out, M, N, N, True)
    first = _area(M, N, (slice(0, 256), slice(0, 256)), (slice(ends[1], ends[1] + 128), slice(6 * 256, 6 * 256 + 128)))
    if blocks == 1:
        assert np.array_equal(written, first)
    else:
        last = _area(M, N, (slice(ends[1] + 896, ends[2]), slice(15 * 256 + 128, N)))   # quarter 63
        assert written[first].all() and written[last].all()
        assert written.sum() <= 3 * 256 * 256 + 2 * 128 * 128
