"""MXFP4 quantizer: where its bytes land. One tile, partial tiles either way; scale buffers that start at any byte;
the places of a tiled scale buffer that belong to no block, and what lies around every buffer, stay as they were."""
import numpy as np
import pytest
import torch

import paper_2506_08027_amd as mx
import scale_layout as sl
from oracle import mxfp4
from paper_2506_08027_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(32, 160), (64, 96), (64, 288), (128, 128), (160, 288), (96, 416), (416, 96)])
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("tiled", [False, True], ids=["rowmajor", "tiled"])
@pytest.mark.parametrize("off", [0, 1])
def test_places(shape, bf16, tiled, off):
    rows, cols = shape
    x = si.fp4_hard_cases(rows, cols, seed=rows + cols)
    x[3 % rows, 5 % cols], x[rows - 1, cols - 1], x[rows - 1, 0] = np.inf, np.nan, -np.inf
    src = si.to_bf16_bits(x) if bf16 else x
    dev = torch.from_numpy(src.view(np.int16) if bf16 else src).cuda()
    dev = dev.view(torch.bfloat16) if bf16 else dev
    lay = mx.SCALES_TILED if tiled else mx.SCALES_ROWMAJOR
    hold, out = {}, {}
    for q, s, r, c in (("q_row", "s_row", rows, cols), ("q_colT", "s_colT", cols, rows)):
        n = mx.mxfp8_scale_bytes(r, c, lay)
        hold[q] = torch.full((32 + r * c // 2,), 0xEE, dtype=torch.uint8, device="cuda")
        hold[s] = torch.full((32 + n,), 0xEE, dtype=torch.uint8, device="cuda")
        out[q] = hold[q][16:16 + r * c // 2].view(r, c // 2)
        out[s] = hold[s][8 + off:8 + off + n]
        if not tiled:
            out[s] = out[s].view(r, c // 32)
    mx.mxfp8_fp4_quantize_ex(dev, mx.BOTH, **out, scale_layout=lay)
    torch.cuda.synchronize()
    for q, s, ref in (("q_row", "s_row", mxfp4.quantize_rowwise), ("q_colT", "s_colT", mxfp4.quantize_colwise)):
        want_q, want_s = ref(src)
        assert np.array_equal(out[q].cpu().numpy(), want_q), q
        got = out[s].cpu().numpy()
        assert np.array_equal(got, sl.tile(want_s, filler=0xEE) if tiled else want_s), s
        for name, first, n in ((q, 16, out[q].numel()), (s, 8 + off, out[s].numel())):
            edge = hold[name].cpu().numpy()
            assert (edge[:first] == 0xEE).all() and (edge[first + n:] == 0xEE).all(), name


@pytest.mark.parametrize("rows", [32, 64, 96])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [mx.SCALES_ROWMAJOR, mx.SCALES_TILED], ids=["rowmajor", "tiled"])
def test_one_copy_is_the_same_as_of_both(rows, dtype, layout):
    x = torch.from_numpy(si.fp4_hard_cases(rows, 2080, seed=rows)).cuda().to(dtype)
    both = mx.fp4_quantize(x, "both", layout)
    for axis, names in (("rowwise", ("q_row", "s_row")), ("colwise", ("q_colT", "s_colT"))):
        one = mx.fp4_quantize(x, axis, layout)
        for name in names:
            if layout == mx.SCALES_TILED and name[0] == "s":
                r, c = (rows, 2080) if name == "s_row" else (2080, rows)
                assert np.array_equal(sl.untile(one[name].cpu().numpy(), r, c // 32), sl.untile(both[name].cpu().numpy(), r, c // 32))
            else:
                assert torch.equal(one[name], both[name])
