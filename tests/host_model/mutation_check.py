"""Sensitivity check of the CPU execution model (test infrastructure; `python tests/host_model/mutation_check.py`,
or tests/test_mutation_checks.py with --runslow). Plants one mistake at a time into a scratch
copy of the product kernels' sources -- a removed barrier, a wait count that is one too loose, a missing wait,
a swizzle mismatch, a prefetch into the wrong buffer or of the wrong K step, a missing ragged-tile clamp, a scale
of another row or step, a wrong output row -- builds the host model from it and runs a few products on that kernel
(one-tile, resident, resident on ragged problems, staged, a rest of tiles as quarters, grouped weight gradients) against the oracle in the scheduling modes (lazy /
eager DMA completion, either wavefront running ahead). Every mutant must be caught, by a wrong, NaN or missing
result or by the model's range check. A second group plants mistakes into the
converters (scale-rule constants, the staging swizzle of the transposed copy, a removed barrier, the infinity patch,
the narrow formats' scale rules) and compares the quantized bytes with the oracle's. Arguments, if any, select the
mutants whose description contains one of them."""
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)
sys.path.insert(0, os.path.dirname(HERE))
import oracle  # noqa: E402
import scale_layout as sl  # noqa: E402

MID = ("                MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB);  // all but this step's requests: A(kt+1) is in LDS\n"
       "                __syncthreads();")
END = ("        MXFP8_WAIT_VMCNT(Cfg::NA);  // everything older than this step's A requests: B(kt+1) is in LDS\n"
       "        __syncthreads();")
PRO = ("        MXFP8_WAIT_VMCNT(0);\n        __syncthreads();\n#pragma unroll\n        for (int i = 0; i < TM; ++i) {\n"
       "            fa[i] = read_frag(lds + Cfg::A_OFF")
MUTANTS = [  # (description, old text, new text): first occurrence, i.e. in the one-tile-per-workgroup kernel
    ("barrier before the last MFMA column removed", MID, MID.replace("\n                __syncthreads();", "")),
    ("barrier at the end of the K step removed", END, END.replace("\n        __syncthreads();", "")),
    ("mid-step wait one request too loose", "MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB);  // all but",
     "MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB + 1);  // all but"),
    ("end-of-step wait one request too loose", "MXFP8_WAIT_VMCNT(Cfg::NA);  // everything older",
     "MXFP8_WAIT_VMCNT(Cfg::NA + 1);  // everything older"),
    ("prologue does not wait for its loads", PRO, PRO.replace("        MXFP8_WAIT_VMCNT(0);\n", "")),
    ("fragment read uses another swizzle than the load", "const int a_off0 = a_row * BK + ((g ^ ((a_row >> 1) & 7)) << 4)",
     "const int a_off0 = a_row * BK + ((g ^ ((a_row >> 2) & 7)) << 4)"),
    ("A prefetch goes to the buffer still in use", "issue_a(a_slot, kt2, cur);", "issue_a(a_slot, kt2, nxt);"),
    ("B prefetch fetches the wrong K step", "const int kt1 = min(kt + 1, KT - 1), kt2", "const int kt1 = min(kt + 2, KT - 1), kt2"),
    ("ragged tile reads past the last row", "a_goff[i] = (uint32_t)min(row, M - 1 - m0) * (uint32_t)K + chunk * 16;",
     "a_goff[i] = (uint32_t)row * (uint32_t)K + chunk * 16;"),
    ("row-major scale dwords land in the wrong 64-row group",
     "                dma_load<4>(as_tile + (kt * SDW + dw) * 4, as_goff[i],\n                            lds_base + Cfg::SA_OFF + buf * Cfg::SA_BYTES + dw * Cfg::BM * 4 + a_grp(i) * 256);",
     "                dma_load<4>(as_tile + (kt * SDW + dw) * 4, as_goff[i],\n                            lds_base + Cfg::SA_OFF + buf * Cfg::SA_BYTES + dw * Cfg::BM * 4 + ((a_grp(i) + 1) % (Cfg::BM / 64)) * 256);"),
    ("epilogue stores to the rows of another wavefront", "const int m = m0 + wm * Cfg::WM + i * 16 + r16;",
     "const int m = m0 + wn * Cfg::WM + i * 16 + r16;"),
]
# the same kinds of mistake in the persistent kernel (last occurrence of the text; run with several tiles per workgroup)
PERSISTENT_MUTANTS = [
    ("persistent: barrier before the last MFMA column removed",
     "                MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB);\n                MXFP8_BARRIER();",
     "                MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB);"),
    ("persistent: end-of-step wait one request too loose", "        MXFP8_WAIT_VMCNT_AND_LDS(Cfg::NA);\n        MXFP8_BARRIER();",
     "        MXFP8_WAIT_VMCNT_AND_LDS(Cfg::NA + 1);\n        MXFP8_BARRIER();"),
    ("persistent: barrier at the end of the K step removed",
     "        MXFP8_WAIT_VMCNT_AND_LDS(Cfg::NA);\n        MXFP8_BARRIER();", "        MXFP8_WAIT_VMCNT_AND_LDS(Cfg::NA);"),
    ("persistent: next tile's B fetched one K step late", "                b_src = next_tile.b;\n", "                b_src = next_tile.b + BK;\n"),
    ("persistent: next tile's first A step fetched from the current tile",
     "                a_src = next_tile.a + (int64_t)(kt + 2 - KT) * BK;", "                a_src = cur_tile.a + (int64_t)(kt + 2 - KT) * BK;"),
    ("persistent: accumulators not cleared between tiles", "                acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};\n        cur_tile = next_tile;",
     "                ;\n        cur_tile = next_tile;"),
    ("persistent: buffer parity not carried across tiles", "            step(par, b_src, bs_src, a_src, as_src, a_lim);\n            par ^= 1;",
     "            step(kt & 1, b_src, bs_src, a_src, as_src, a_lim);\n            par ^= 1;"),
]
# ragged problems on the resident kernel (three by three tiles on two workgroups, the last row and column moved back)
RAGGED_MUTANTS = [
    ("ragged: A scales of the next tile read at the current tile's offset", "as_off = kt + 2 < KT ? cur_tile.as_off : next_tile.as_off;",
     "as_off = cur_tile.as_off;"),
    ("ragged: B scales of the next tile read at the current tile's offset", "bs_off = kt + 1 < KT ? cur_tile.bs_off : next_tile.bs_off;",
     "bs_off = cur_tile.bs_off;"),
    ("ragged: last row of tiles not moved back", "t.m0 = RAGGED ? min(tm * Cfg::BM, M - Cfg::BM) : tm * Cfg::BM;", "t.m0 = tm * Cfg::BM;"),
    ("ragged: tiled scales of a moved tile as if it began a 64-row group", "            if constexpr (RAGGED) {\n                const int row = first + lane;",
     "            if constexpr (false) {\n                const int row = first + lane;"),
    ("ragged: first own row of a moved tile not stored", "(m >= cur_tile.row_lo &&", "(m > cur_tile.row_lo - (cur_tile.row_lo == 0) &&"),
]
STEP_BARRIER = ("                MXFP8_BARRIER();\n                MXFP8_FENCE();\n            }\n            MXFP8_PIN();")
STAGED_MUTANTS = [  # gemm_staged_tiles.h
    ("staged: prologue wait one request too loose", "MXFP8_WAIT_VMCNT_AND_LDS((S - 1) * L);", "MXFP8_WAIT_VMCNT_AND_LDS((S - 1) * L + 1);"),
    ("staged: wait of a step one request too loose", "MXFP8_WAIT_VMCNT_AND_LDS((S - 2) * L);", "MXFP8_WAIT_VMCNT_AND_LDS((S - 2) * L + 1);"),
    ("staged: waits of the last steps one step too loose", "wait_tail<S - 2, L>(left - 1);", "wait_tail<S - 2, L>(left);"),
    ("staged: barrier of a step removed", STEP_BARRIER, STEP_BARRIER.replace("                MXFP8_BARRIER();\n", "")),
    ("staged: request into the next ring slot", "issue(t, kt + S, slot);", "issue(t, kt + S, next);"),
    ("staged: request of the wrong K step", "issue(t, kt + S, slot);", "issue(t, kt + S - 1, slot);"),
    ("staged: fragments read from the slot of the step that runs", "read_piece(p, kt + 1, next, set ^ 1);", "read_piece(p, kt + 1, slot, set ^ 1);"),
    ("staged: odd first step computed twice", "            step(0, 1, S);\n            kt = 1;", "            step(0, 1, S);"),
    ("staged: quarters of row-major scales out of order", "ahead % SPG * SDW);", "(ahead + 1) % SPG * SDW);"),
    ("staged: row-major scales of another step of the group", "(kt % SPG) * (4 * SDW)", "((kt + 1) % SPG) * (4 * SDW)"),
    ("staged: scales of a tile that begins inside a 64-row group", "const int sa_row = (TILED ? m0 & 63 : 0) + a_row,", "const int sa_row = a_row,"),
    ("staged: ragged tile reads past the last row", "goff[i] = (uint32_t)min(row, (is_a ? M - m0 : N - n0) - 1) * (uint32_t)K", "goff[i] = (uint32_t)row * (uint32_t)K"),
    ("staged: no barrier before the next tile's requests", "            __syncthreads();  // the next tile's requests go where the rows were staged", "            ;"),
]
# a rest of 256x256 tiles as quarters: the second launch of a plain product, the end of a grouped one's
QUARTER_MUTANTS = [
    ("quarters: the first tiles instead of the rest", "tile_of_block(done + (tile >> 2), whole_tiles", "tile_of_block(tile >> 2, whole_tiles"),
    ("quarters: two of four computed twice", "n0 = tile_n * 256 + (tile & 1) * 128;", "n0 = tile_n * 256 + (tile >> 1 & 1) * 128;"),
]
REST_MUTANTS = [
    ("grouped rest: rows counted from the first expert's", "m0 = first_row + tile_m * 256", "m0 = tile_m * 256"),
    ("grouped rest: rows behind the expert's end stored", "M = at.end;", "M = M_all;"),
    ("grouped rest: weights of the first expert", "b_q += at.expert * groups.b_group_bytes;", ""),
]
# grouped weight gradients on resident workgroups, first occurrence in gemm.hip
WGRAD_MUTANTS = [
    ("wgrad: A requests two steps ahead stay in the next tile", "const bool a_next = kt + 2 - steps < next_tile.steps;", "const bool a_next = true;"),
    ("wgrad: B scales of the next tile read at the current tile's offset", "bs_off = b_here ? cur_tile.bs_off : next_tile.bs_off;", "bs_off = cur_tile.bs_off;"),
    ("wgrad: B of every expert from the first step on", "            t.b += first_step * BK;\n", ""),
    ("wgrad: second step of a one-step tile fetched past its expert", "        if (cur_tile.steps == 1) {", "        if (false) {"),
    ("wgrad: experts without a step not cleared", "(int64_t)i * 16) = make_uint4(0, 0, 0, 0);", "(int64_t)i * 16) = make_uint4(1, 0, 0, 0);"),
    ("wgrad: experts of the same number of steps share a place", "(uint32_t)steps1 * kMostKExperts + (kMostKExperts - 2 - 2 * lane)", "(uint32_t)steps1 * kMostKExperts + (kMostKExperts - 1 - 2 * lane)"),
    ("wgrad: tiles lost behind rounds that workgroups sit out", "min(max(round - 1, 0), skipped) * busy", "min(round, skipped) * busy"),
    ("wgrad: rounds that go backwards counted from the end of the whole round", "(round & 1 ? width - 1 - place : place)", "(round & 1 ? (int)gridDim.x - 1 - place : place)"),
]
MODES = [{}, {"WAVESIM_ORDER": "down"}, {"WAVESIM_DMA": "eager"}, {"WAVESIM_DMA": "eager", "WAVESIM_ORDER": "down"}]


def build(work, text, name="gemm.hip"):
    csrc = os.path.join(work, "csrc")
    shutil.copytree(os.path.join(ROOT, "paper_2506_08027_amd", "csrc"), csrc)
    open(os.path.join(csrc, name), "w").write(text)
    inc = os.path.join(ROOT, "include", "mxfp8.h")
    for name, path in (("api.hip", csrc), ("driver.cpp", work)):
        src = os.path.join(csrc if name == "api.hip" else HERE, name)
        text = open(src).read().replace('"../../include/mxfp8.h"', f'"{inc}"').replace('"wavesim.h"', f'"{HERE}/wavesim.h"')
        open(os.path.join(path, name), "w").write(text)
    binary = os.path.join(work, "hostmodel")
    cmd = ["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-x", "c++", "-I", os.path.join(HERE, "shim"), "-O0",
           "-Wno-unknown-pragmas", "-Wno-psabi", "-o", binary, os.path.join(work, "driver.cpp")]
    cmd += [os.path.join(csrc, f) for f in sorted(os.listdir(csrc)) if f.endswith(".hip")]
    subprocess.run(cmd, check=True, capture_output=True)
    return binary


# kernel -> [(M, N, K steps, tiled scales, bound on workgroups, units, simulated workgroups or 0 = all)]
CASES = {
    "one-tile": [(200, 136, 3, False, 0, 256, 0), (130, 129, 2, True, 0, 256, 0), (2047, 4095, 3, False, 0, 256, 2)],
    # 6 small tiles on 2 workgroups, 128 large tiles on 64: K = 3 steps (odd: parity flips per tile)
    "resident": [(256, 384, 3, False, 2, 256, 0), (2048, 4096, 3, False, 64, 256, 2)],
    "ragged": [(760, 744, 5, True, 0, 2, 0)],
    # 32x32 tiles in both scale layouts, several 128x128 tiles per workgroup
    "staged": [(70, 72, 9, False, 0, 256, 0), (70, 72, 6, True, 0, 256, 0), (384, 256, 12, False, 2, 256, 0), (384, 384, 11, True, 3, 256, 0)],
}


def caught(binary, work, kernel):
    for M, N, steps, tiled, bound, units, blocks in CASES[kernel]:
        K = steps * 128
        rng = np.random.default_rng(M + N)
        a = rng.standard_normal((M, K)).astype(np.float32) * np.exp2(rng.integers(-6, 7, (M, 1))).astype(np.float32)
        b = (rng.standard_normal((N, K)) * 0.02).astype(np.float32) * np.exp2(rng.integers(-6, 7, (N, 1))).astype(np.float32)
        ops = oracle.quantize_rowwise(a) + oracle.quantize_rowwise(b)
        names = []
        for n, v in zip(("aq", "as", "bq", "bs"), ops):
            names.append(os.path.join(work, n + ".bin"))
            (sl.tile(v, filler=0xFF) if tiled and n.endswith("s") else v).tofile(names[-1])
        out = os.path.join(work, "c.bin")
        case = os.path.join(work, "case.txt")
        open(case, "w").write(f"gemm 0 {M} {N} {K} f32 {N} {' '.join(names)} {out}" + (" tiled" if tiled else "") +
                              (f" wg={bound}" if bound else "") + "\n")
        for mode in MODES:
            env = dict(os.environ, WAVESIM_BLOCKS=str(blocks or "all"), WAVESIM_CUS=str(units), **mode)
            r = subprocess.run([binary, case], capture_output=True, text=True, env=env)
            if r.returncode != 0:
                return f"model stopped: {(r.stderr.strip().splitlines() or ['exit code ' + str(r.returncode)])[-1][:100]}"
            c = np.fromfile(out, np.uint32).reshape(M, N)
            written = c != 0xA5A5A5A5
            if not blocks and not written.all():
                return f"{(~written).sum()} results missing at {M}x{N}x{K} in mode {mode or 'default'}"
            rows = np.unique(np.nonzero(written)[0])
            ref, absum = oracle.gemm_rows(*ops, rows)
            val = c.view(np.float32)[rows]
            w = written[rows]
            if np.isnan(val[w]).any() or (np.abs(val - ref)[w] > (max(steps, 2) * 2.0 ** -24 * absum + 1e-300)[w]).any():
                return f"wrong result at {M}x{N}x{K} in mode {mode or 'default'}"
    return None


def caught_quarters(binary, work, kernel):
    """Every quarter of the second launch of a plain product (nine ragged tiles on eight units)."""
    M, N, K = 700, 760, 28 * 128
    rng = np.random.default_rng(7)
    ops = oracle.quantize_rowwise(rng.standard_normal((M, K)).astype(np.float32)) + oracle.quantize_rowwise(rng.standard_normal((N, K)).astype(np.float32))
    out, names = os.path.join(work, "c.bin"), [os.path.join(work, n + ".bin") for n in ("aq", "as", "bq", "bs")]
    for path, v in zip(names, ops):
        (sl.tile(v, filler=0xFF) if path.endswith("s.bin") else v).tofile(path)
    case = os.path.join(work, "case.txt")
    open(case, "w").write(f"gemm 0 {M} {N} {K} f32 {N} {' '.join(names)} {out} tiled\n")
    r = subprocess.run([binary, case], capture_output=True, text=True, env=dict(os.environ, WAVESIM_CUS="8", WAVESIM_ONLY="1"))
    if r.returncode != 0:
        return f"model stopped: {(r.stderr.strip().splitlines() or ['exit code ' + str(r.returncode)])[-1][:100]}"
    c = np.fromfile(out, np.uint32).reshape(M, N)
    want = np.zeros((M, N), bool)
    want[512:, 512:] = True
    if not np.array_equal(c != 0xA5A5A5A5, want):
        return "quarters missing, or others written"
    ref, absum = oracle.gemm_rows(*ops, np.arange(512, M))
    bad = np.abs(c.view(np.float32)[512:, 512:] - ref[:, 512:]) > (K // 128 * 2.0 ** -24 * absum + 1e-300)[:, 512:]
    return "wrong result" if bad.any() else None


def caught_grouped(binary, work, kernel):
    """grouped rest: three workgroups of a product of three experts whose last sixteen tiles are quarters; wgrad: experts of 0 .. 10 steps,
    whole and ragged tiles, workgroups that sit out a round."""
    rng = np.random.default_rng(8)
    rest = kernel == "grouped rest"
    for M, N, steps, units, tiled, blocks in ([(2048, 4096, 16, 128, False, 3)] if rest else [(264, 520, [1, 1, 0, 2, 0, 3, 1, 1] + [0] * 56, 5, True, 0),
                                                                                           (512, 256, [1, 1, 0, 10, 1, 1, 1, 1] + [0] * 56, 5, False, 0)]):
        K = steps * 128 if rest else sum(steps) * 128
        ends = [400, 1003, 2001] if rest else [int(e) * 128 for e in np.cumsum(steps)]
        a = oracle.quantize_rowwise(rng.standard_normal((M, K)).astype(np.float32) * np.exp2(rng.integers(-6, 7, (M, 1))).astype(np.float32))
        bs = [oracle.quantize_rowwise((rng.standard_normal((N, K)) * 0.02).astype(np.float32) * np.exp2(rng.integers(-6, 7, (N, 1))).astype(np.float32))
              for _ in range(len(ends) if rest else 1)]
        ops = a + ((np.stack([q for q, _ in bs]), np.stack([s for _, s in bs])) if rest else bs[0])
        scales = (lambda s: np.concatenate([sl.tile(x, filler=0xFF).ravel() for x in (s if s.ndim == 3 else [s])])) if tiled else (lambda s: s)
        names = [os.path.join(work, n + ".bin") for n in ("aq", "as", "bq", "bs", "ends")]
        for path, v in zip(names, (ops[0], scales(ops[1]), ops[2], scales(ops[3]), np.asarray(ends, np.int32))):
            v.tofile(path)
        out, case, bf16 = os.path.join(work, "c.bin"), os.path.join(work, "case.txt"), not tiled and not rest
        open(case, "w").write(f"{'gemmgrp' if rest else 'gemmgrpk'} {M} {N} {K} {'bf16' if bf16 else 'f32'} {N} {len(ends)} {' '.join(names)} {out}" + (" tiled" if tiled else "") + "\n")
        for mode in MODES[:1] if rest else MODES[::3]:
            r = subprocess.run([binary, case], capture_output=True, text=True,
                               env=dict(os.environ, WAVESIM_CUS=str(units), WAVESIM_BLOCKS=str(blocks or "all"), **mode))
            if r.returncode != 0:
                return f"model stopped: {(r.stderr.strip().splitlines() or ['exit code ' + str(r.returncode)])[-1][:100]}"
            raw = np.fromfile(out, np.uint16 if bf16 else np.uint32).reshape(-1, N)
            written = raw != (0xA5A5 if bf16 else 0xA5A5A5A5)
            val = (raw.astype(np.uint32) << 16).view(np.float32) if bf16 else raw.view(np.float32)
            ref, absum = (oracle.grouped_gemm if rest else oracle.grouped_gemm_wgrad)(*ops, ends)
            ref, absum = np.reshape(ref, raw.shape), np.reshape(absum, raw.shape)
            owned = ~np.isnan(ref)
            if (written & ~owned).any() or not (written.all() if not rest else written[ends[1]:ends[1] + 128, 6 * 256:6 * 256 + 128].all()):
                return "rows missing, or others written"
            tol = K // 128 * 2.0 ** -24 * absum + (2.0 ** -8 * np.abs(ref) if bf16 else 0.0) + 1e-300
            if np.isnan(val[written]).any() or (np.abs(val - ref)[written] > tol[written]).any():
                return f"wrong result at {M}x{N} in mode {mode or 'default'}"
    return None


# mistakes in the converters: (description, source file, old text, new text), first occurrence
QUANT_MUTANTS = [
    ("quantizer: FP32 scale rule carries at 1.875 instead of 1.75", "mxfp8_device.h",
     "(abs_bits + 0x1FFFFFu) >> 23) - 8", "(abs_bits + 0x0FFFFFu) >> 23) - 8"),
    ("quantizer: BF16 scale rule carries at 1.875 instead of 1.75", "mxfp8_device.h",
     "(abs_bits16 + 0x1Fu) >> 7) - 8", "(abs_bits16 + 0x0Fu) >> 7) - 8"),
    ("quantizer: staging swizzle of the transposed copy differs from the write-out's", "quantize_tile.h",
     "const int slot16 = (lrow0 >> 4) ^ (cc & 7);", "const int slot16 = (lrow0 >> 4) ^ ((cc + 1) & 7);"),
    ("quantizer: barrier between staging and write-out removed", "quantize_tile.h",
     "    __syncthreads();\n\n    // ---- write-out of the staged pieces", "\n    // ---- write-out of the staged pieces"),
    ("quantizer: infinities keep the converter's NaN code in the row copy", "quantize_tile.h",
     "f0 |= inf_byte<BF16, MODE>(elem_at<BF16>(x[i], j), (q0 >> (8 * j)) & 0xFFu) << (8 * j);",
     "f0 |= ((q0 >> (8 * j)) & 0xFFu) << (8 * j);"),
    ("quantizer: MXFP4 scale rule carries at 1.75 instead of 1.5", "mxfp4.hip",
     "(abs_bits + 0x3FFFFFu) >> 23) - 2", "(abs_bits + 0x1FFFFFu) >> 23) - 2"),
    ("quantizer: MXFP4 of BF16 sources, the other column of a pair in the column copy", "mxfp4.hip", "(j & 1) ? 0x07060302u : 0x05040100u", "(j & 1) ? 0x05040100u : 0x07060302u"),
    ("quantizer: MXFP4 of BF16 sources, maxima of the other column of a pair", "mxfp4.hip", "(j & 1) ? (cm[j >> 1] & 0xFFFF0000u) >> 1", "!(j & 1) ? (cm[j >> 1] & 0xFFFF0000u) >> 1"),
    ("quantizer: MXFP4 blocks with a NaN keep the converter's codes", "mxfp4.hip", "    if (sb == 0xFFu)\n        return make_uint4(0, 0, 0, 0);", ""),
    ("quantizer: MXFP6 scale exponent one too large", "mxfp6.hip",
     "(0x7FFFFFu - F::TOP_FRAC)) >> 23) - F::EMAX;", "(0x7FFFFFu - F::TOP_FRAC)) >> 23) - F::EMAX + 1;"),
]


def caught_quant(binary, work):
    """Quantizes the tiny configuration (every special block) as FP32 and as BF16 along both axes, and hard cases of
    the narrow formats, and compares every output byte with the oracle."""
    from oracle import mxfp4, mxfp6
    from paper_2506_08027_amd import synth_inputs as si
    x = si.tiny_with_specials(256, seed=0)
    cases = []
    for bf16 in (False, True):
        src = si.to_bf16_bits(x) if bf16 else x
        cases.append((f"quantize {'bf16' if bf16 else 'f32'} 256 256 256 3", src,
                      (oracle.quantize_rowwise(src), oracle.quantize_colwise(src))))
    h4 = si.fp4_hard_cases(160, 96, seed=12)
    for src in (h4, si.to_bf16_bits(h4)):
        cases.append((f"quantfp4 {'f32' if src is h4 else 'bf16'} 160 96 96 3", src, (mxfp4.quantize_rowwise(src), mxfp4.quantize_colwise(src))))
    h6 = si.fp6_hard_cases(160, 96, seed=12, top=7.5)
    cases.append(("quantfp6 f32 160 96 96 3 0", h6, (mxfp6.quantize_rowwise(h6, "e2m3"), mxfp6.quantize_colwise(h6, "e2m3"))))
    for head, src, ((q, s), (qT, sT)) in cases:
        path = os.path.join(work, "src.bin")
        np.ascontiguousarray(src).tofile(path)
        prefix = os.path.join(work, "o")
        case = os.path.join(work, "case.txt")
        open(case, "w").write(f"{head} {path} {prefix}\n")
        r = subprocess.run([binary, case], capture_output=True, text=True)
        if r.returncode != 0:
            return f"model stopped: {r.stderr.strip().splitlines()[-1][:100]}"
        for suffix, want in ((".q_row", q), (".s_row", s), (".q_colT", qT), (".s_colT", sT)):
            if not np.array_equal(np.fromfile(prefix + suffix, np.uint8), want.ravel()):
                return f"wrong bytes in {suffix[1:]} of '{head}'"
    return None


def main():
    csrc = os.path.join(ROOT, "paper_2506_08027_amd", "csrc")
    # (description, source file, old text, new text, kernel whose cases are run; None: the converters'), first occurrence
    # of the text, in the resident kernel the last one (the one-tile kernel before it has the same)
    todo = [(f"(unmutated source, {kernel}: must pass)", "gemm.hip", "", "", kernel) for kernel in CASES]
    todo += [(desc, "gemm.hip", old, new, "one-tile") for desc, old, new in MUTANTS]
    todo += [(desc, "gemm.hip", old, new, "resident") for desc, old, new in PERSISTENT_MUTANTS]
    todo += [(desc, "gemm.hip", old, new, "ragged") for desc, old, new in RAGGED_MUTANTS]
    todo += [(desc, "gemm_staged_tiles.h", old, new, "staged") for desc, old, new in STAGED_MUTANTS]
    todo += [(f"(unmutated source, {kernel}: must pass)", "gemm.hip", "", "", kernel) for kernel in ("quarters", "grouped rest", "wgrad")]
    todo += [(desc, "gemm_staged_tiles.h", old, new, "quarters") for desc, old, new in QUARTER_MUTANTS]
    todo += [(desc, "gemm_staged_tiles.h", old, new, "grouped rest") for desc, old, new in REST_MUTANTS]
    todo += [(desc, "gemm.hip", old, new, "wgrad") for desc, old, new in WGRAD_MUTANTS]
    todo += [("(unmutated converters: must pass)", "gemm.hip", "", "", None)] + [m + (None,) for m in QUANT_MUTANTS]
    for desc, name, old, new, kernel in todo:   # every pattern must still be in the source: a stale one would test nothing
        assert old == "" or old in open(os.path.join(csrc, name)).read(), desc
    only = sys.argv[1:]
    todo = [m for m in todo if not only or any(o in m[0] for o in only)]

    def run(mutant):
        desc, name, old, new, kernel = mutant
        text = open(os.path.join(csrc, name)).read()
        if old:
            at = (text.rindex if kernel == "resident" else text.index)(old)
            text = text[:at] + new + text[at + len(old):]
        work = tempfile.mkdtemp(prefix="kmut_")
        try:
            binary = build(work, text, name)
            look = {None: lambda b, w, k: caught_quant(b, w), "quarters": caught_quarters, "grouped rest": caught_grouped, "wgrad": caught_grouped}
            how = look.get(kernel, caught)(binary, work, kernel)
        finally:
            shutil.rmtree(work, ignore_errors=True)
        ok = (how is None) if old == "" else (how is not None)
        print(("ok      " if ok else "PROBLEM ") + desc + (f" -> {how}" if how else ""), flush=True)
        return ok

    with ThreadPoolExecutor(max(1, min(6, (os.cpu_count() or 2) - 1))) as pool:
        results = list(pool.map(run, todo))
    planted = sum(m[2] != "" for m in todo)
    print(f"{len(results) - results.count(False)} of {len(results)} as expected ({planted} planted mistakes)")
    sys.exit(0 if all(results) else 1)


if __name__ == "__main__":
    main()
