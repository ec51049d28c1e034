"""The plain products on every kernel and tile they can take (tests/route_cases.py; tests/test_host_model_routes.py holds the
launches to that table), on the hardware. Each output element goes through the same sequence of matrix instructions on all of
them, so the product must equal, bit for bit, the same product computed from slices of a few rows of A (staged tiles of 32 or
64 rows); sampled rows are held to the oracle as well."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2506_08027_amd as mx
import scale_layout as sl
from oracle import mxfp4
from paper_2506_08027_amd import synth_inputs as si
from route_cases import K_STEP, ROUTES

pytestmark = [pytest.mark.gpu, pytest.mark.skipif("MXFP8_HOSTMODEL_LIB" in os.environ, reason="sizes for the hardware")]
SLICE = 40   # rows, no multiple of a tile


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _operands(fmt, M, N, K, seed):
    """Operands of the format on the host: element bytes (finite codes) and scale bytes; BF16: bit patterns."""
    rng = np.random.default_rng(seed)
    if fmt == "bf16":
        return tuple(v for rows in (M, N) for v in (si.to_bf16_bits(rng.standard_normal((rows, K), dtype=np.float32)), None))
    width, mask = (K // 2, 0xFF) if fmt == "fp4" else (K, 0xF7)
    return tuple(v for rows in (M, N) for v in (rng.integers(0, 256, (rows, width), dtype=np.uint8) & np.uint8(mask),
                                                rng.integers(120, 131, (rows, K // 32), dtype=np.uint8)))


def _product(fmt, ops, c, tiled, bound=0):
    a_q, a_s, b_q, b_s = ops
    if fmt == "bf16":
        return mx.mxfp8_gemm_bf16(a_q, b_q, c, max_workgroups=bound)
    lay = mx.SCALES_TILED if tiled else mx.SCALES_ROWMAJOR
    if fmt == "fp4":
        return mx.mxfp8_fp4_gemm_ex("fprop", a_q, a_s, b_q, b_s, c, lay, bound)
    if fmt == "e5m2":
        return mx.mxfp8_gemm_mode_ex("dgrad", a_q, a_s, mx.E5M2, b_q, b_s, mx.E4M3, c, lay, bound)
    return mx.mxfp8_gemm_ex("fprop", a_q, a_s, b_q, b_s, c, lay, bound)


def _reference(fmt, ops, rows):
    """Oracle's product of the given rows, and sum|a b|."""
    a_q, a_s, b_q, b_s = ops
    if fmt == "bf16":
        return oracle.matmul_nt_bf16(np.ascontiguousarray(a_q[rows]), b_q)
    if fmt == "fp4":
        return mxfp4.gemm(a_q[rows], a_s[rows], b_q, b_s)
    if fmt == "e5m2":
        return oracle.gemm_mode(a_q[rows], a_s[rows], "e5m2", b_q, b_s, "e4m3")
    return oracle.gemm_rows(a_q, a_s, b_q, b_s, rows)


@pytest.mark.parametrize("case", ROUTES, ids=lambda c: "-".join([c[1][0], f"{c[1][1]}x{c[1][2]}"] + [str(int(v)) if not isinstance(v, str) else v for v in c[0]]))
def test_product_is_the_same_on_every_route(case):
    (fmt, M, N, steps, bf16, pad, tiled, bound), _ = case
    K = steps * K_STEP[fmt]
    host = _operands(fmt, M, N, K, seed=M + steps)
    dtype, bits = (torch.bfloat16, torch.int16) if bf16 else (torch.float32, torch.int32)
    scales = (lambda s: _dev(sl.tile(s, filler=0xFF))) if tiled else _dev
    to_dev = (lambda t: _dev(t.view(np.int16)).view(torch.bfloat16)) if fmt == "bf16" else _dev
    b_q, b_s = to_dev(host[2]), None if fmt == "bf16" else scales(host[3])
    full = torch.full((M, N + pad), -3.0, dtype=dtype, device="cuda")
    c = full[:, :N]
    _product(fmt, (to_dev(host[0]), None if fmt == "bf16" else scales(host[1]), b_q, b_s), c, tiled, bound)
    sliced = torch.empty((M, N), dtype=dtype, device="cuda")
    for m in range(0, M, SLICE):
        part = slice(m, min(m + SLICE, M))
        _product(fmt, (to_dev(host[0][part]), None if fmt == "bf16" else scales(host[1][part]), b_q, b_s), sliced[part], tiled)
    torch.cuda.synchronize()
    assert torch.equal(c.contiguous().view(bits), sliced.view(bits))
    assert (full[:, N:] == -3.0).all()
    rows = np.unique(np.linspace(0, M - 1, 7).astype(int))
    ref, absum = _reference(fmt, host, rows)
    got = c[torch.from_numpy(rows).cuda()].to(torch.float64).cpu().numpy()
    # FP8 products are cut off inside groups of eight (2^-10 of sum|ab| bounds it), the others are FP32 sums: K additions of
    # 2^-24 each at worst, far below 2^-16 for these K; one BF16 rounding of the output
    tol = (2.0 ** -10 if fmt in ("fp8", "e5m2") else 2.0 ** -16) * absum + (2.0 ** -8 * np.abs(ref) if bf16 else 0.0) + 1e-300
    assert (np.abs(got - ref) <= tol).all()
