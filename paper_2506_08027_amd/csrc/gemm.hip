// Block-scaled MXFP8 GEMM for gfx950: C[M x N] = A[M x K] * B[N x K]^T, both operands K-contiguous
// E4M3 with one UE8M0 scale per 32 elements of K, FP32 accumulation (Section 2, Appendix A.3).
// The same kernel serves the forward, activation-gradient and weight-gradient products of a
// linear layer (Section 3.2, Figure 2): the column-wise quantized copies are stored transposed,
// which makes every one of them a K-contiguous "NT" product.
//
// Instruction. v_mfma_scale_f32_16x16x128_f8f6f4 multiplies a 16x128 by a 128x16 FP8 tile and
// applies, per operand, one scale byte per row and per 32-wide K block. Register layout (found by
// one-hot probing on the hardware): lane l = 16*g + r holds row r of its operand; its eight
// dwords hold K = 16g..16g+15 followed by K = 64+16g..64+16g+15; the scale operand of lane
// (r, g) is the scale of row r for K block g (K = 32g..32g+31), taken from byte op_sel of the
// register. The result register v of lane (r, g) is D[4g + v][r].
// The kernel feeds B rows as the first operand and A rows as the second, so a lane ends up with
// four consecutive n of one m: the epilogue is one 128-bit store per 16x16 tile and lane.
//
// Tiling. A workgroup of WAVES_M x WAVES_N wavefronts computes a BM x BN tile of C, K in steps of
// 128 bytes (= one MFMA, four scale blocks). A and B tiles and one dword of scale bytes per row
// and step go from global memory straight into LDS (global_load_lds_dword{,x4}: no staging
// registers), two LDS buffers per operand; the software pipeline is described at the step lambda
// of the kernel. LDS rows are 128 bytes; the 16-byte chunk index is XORed with (row/2)%8 so that
// the 16 lanes of a fragment read hit 16 different bank groups. A direct-to-LDS load writes lane l
// of a wavefront to LDS offset 16*l, so the swizzle is applied on the global side: each lane
// fetches the chunk that belongs at its slot.
//
// Other operand formats on the same kernels (GemmCfg's FMT): plain BF16 operands for the product of the
// simulated path (two 16x16x32 BF16 instructions per K step and tile pair, no scales), and MXFP4 operands
// (two E2M1 codes per byte: a 128-byte K step is 256 elements, i.e. two 4-bit scaled instructions and two scale
// dwords per row). With 4-bit elements the instruction takes dwords 0..3 only, lane (r, g) holds K =
// 32g..32g+31 of row r and its own scale byte applies to them (pinned on the hardware by a test that runs
// single instructions on registers taken from memory).
#include <algorithm>
#include <type_traits>
#include "gemm_device.h"
#include "gemm_staged.h"
#include "quantize_tile.h"

namespace mxfp8 {

hipError_t launch_quantize(const void *src, bool bf16, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *q_row, uint8_t *s_row,
                           uint8_t *q_colT, uint8_t *s_colT, bool tiled_scales, int mode, hipStream_t stream);  // quantize.hip

// A_E5M2 / B_E5M2 (kFmtFp8 only): the elements of that operand are E5M2 instead of E4M3 (Section 3.2.2 compares the
// two per tensor type); nothing but the format fields of the matrix instruction changes.
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int FMT_ = kFmtFp8, bool A_E5M2_ = false, bool B_E5M2_ = false> struct GemmCfg {
    static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
    static constexpr int FMT = FMT_;
    static constexpr bool A_E5M2 = A_E5M2_, B_E5M2 = B_E5M2_, ALL_E4M3 = FMT_ == kFmtFp8 && !A_E5M2_ && !B_E5M2_;
    static_assert(FMT_ == kFmtFp8 || (!A_E5M2_ && !B_E5M2_), "element formats belong to the MXFP8 product");
    static constexpr bool SCALED = FMT_ != kFmtBf16;
    static constexpr int SDW = FMT_ == kFmtFp4 ? 2 : 1;     // scale dwords per operand row and K step
    static constexpr int SBLK = FMT_ == kFmtFp4 ? 16 : 32;  // operand bytes per scale block
    static constexpr int WAVES = WAVES_M * WAVES_N;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wavefront tile
    static constexpr int TM = WM / 16, TN = WN / 16;            // MFMA tiles per wavefront
    static constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK;
    // LDS map: A[2] | B[2] | A scales[2] | B scales[2]; a scale buffer holds, for each of the SDW scale dwords of
    // a K step, one dword (4 scale bytes) per tile row: [dword][row][4]
    static constexpr int SA_BYTES = BM * 4 * SDW, SB_BYTES = BN * 4 * SDW;
    static constexpr int A_OFF = 0, B_OFF = 2 * A_BYTES, SA_OFF = B_OFF + 2 * B_BYTES, SB_OFF = SA_OFF + 2 * SA_BYTES;
    static constexpr int LDS_BYTES = SB_OFF + 2 * SB_BYTES;
    static constexpr int LDS_BYTES_PERSISTENT = LDS_BYTES + WAVES * kStageBytes;  // + the epilogue's staging areas
    // one direct-to-LDS instruction moves 8 rows x 128 bytes (or 64 scale dwords) per wavefront
    static constexpr int A_LOADS = BM / 8 / WAVES, B_LOADS = BN / 8 / WAVES;
    static constexpr int SA_LOADS = SCALED ? SDW * ((BM / 64 + WAVES - 1) / WAVES) : 0, SB_LOADS = SCALED ? SDW * ((BN / 64 + WAVES - 1) / WAVES) : 0;
    static constexpr int NA = A_LOADS + SA_LOADS, NB = B_LOADS + SB_LOADS;  // DMA slots per step
    static_assert(BM % (8 * WAVES) == 0 && BN % (8 * WAVES) == 0, "tile rows per wavefront");
    static_assert(BM % 64 == 0 && BN % 64 == 0, "scale rows per instruction");
    static_assert(NB <= 2 * TM, "the B loads of the next step are issued with the MFMAs of the first column");
    static_assert(NA + NB < 64, "wait-count immediate");
};

// The kernel. LDS holds two A buffers, two B buffers and their scale dwords; the software pipeline
// is described at the step lambda below.
// KGROUPED (Appendix A.4, weight gradient of a mixture-of-experts layer): the reduction axis is the token
// axis, sorted by expert; expert e owns K range [group_ends[e-1], group_ends[e]) of both operands and gets its
// own output [M x N], `M * ldc` elements after the previous expert's. Workgroup = (expert, tile); the K range
// comes from device memory, is clamped to [previous end, K] and cut down to whole K steps (ends have to be
// multiples of 128 tokens); an expert without tokens stores zeros.
template <class Cfg, bool OUT_BF16, bool TILED, bool KGROUPED = false>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_kernel(
    const uint8_t *__restrict__ a_q, const uint8_t *__restrict__ a_s, const uint8_t *__restrict__ b_q,
    const uint8_t *__restrict__ b_s, int M, int N, int K, uint8_t *__restrict__ c_all, int64_t ldc_bytes,
    int tiles_m, int tiles_n, bool vec_store, GemmGroups groups)
{
    MXFP8_DYNAMIC_LDS(lds);
    constexpr int TM = Cfg::TM, TN = Cfg::TN;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform: lives in an SGPR
    const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;
    const int r16 = lane & 15, g = lane >> 4;

    int tile_m, tile_n;
    int k0 = 0, k_len = K;  // the K range this workgroup reduces over
    uint8_t *c = c_all;
    if constexpr (KGROUPED) {
        const int per_expert = tiles_m * tiles_n;
        const int e = (int)blockIdx.x / per_expert;
        int prev = 0, end = 0;
        for (int i = 0; i <= e; ++i) {
            prev = end;
            end = min(max(groups.ends[i], prev), K);
        }
        k0 = prev / BK * BK;
        k_len = max(end / BK * BK - k0, 0);
        c += (int64_t)e * M * ldc_bytes;
        tile_of_block((int)blockIdx.x - e * per_expert, per_expert, tiles_m, tiles_n, tile_m, tile_n);
    } else {
        tile_of_block(blockIdx.x, gridDim.x, tiles_m, tiles_n, tile_m, tile_n);
    }
    const int m0 = tile_m * Cfg::BM, n0 = tile_n * Cfg::BN;
    // K is the length of an operand row in BYTES (= elements for MXFP8, 2 x elements for BF16 operands)
    static_assert(!KGROUPED || Cfg::ALL_E4M3, "grouped products take MXFP8-E4M3 operands");
    const int nkb = K / Cfg::SBLK;  // scale bytes per row
    const int KT = k_len / BK;      // steps of this workgroup
    const int KT_row = K / BK;   // steps in a whole operand row (the pitch of the tiled scale layout)

    // ---- global -> LDS addressing: wavefront w owns 8-row groups w*LOADS.. of each tile; one
    // instruction fills 8 consecutive rows, lane l lands at row l/8, physical chunk l%8, and
    // fetches the logical chunk that the XOR swizzle stores there. Offsets are relative to the
    // tile origin (32-bit: a tile spans at most 256 rows of K bytes).
    const int ld_r = lane >> 3, ld_c = lane & 7;
    uint32_t a_goff[Cfg::A_LOADS], b_goff[Cfg::B_LOADS], as_goff[Cfg::SA_LOADS + 1], bs_goff[Cfg::SB_LOADS + 1];
#pragma unroll
    for (int i = 0; i < Cfg::A_LOADS; ++i) {
        const int row = (wave * Cfg::A_LOADS + i) * 8 + ld_r;
        const int chunk = ld_c ^ ((row >> 1) & 7);
        a_goff[i] = (uint32_t)min(row, M - 1 - m0) * (uint32_t)K + chunk * 16;  // ragged tiles re-read a valid row
    }
#pragma unroll
    for (int i = 0; i < Cfg::B_LOADS; ++i) {
        const int row = (wave * Cfg::B_LOADS + i) * 8 + ld_r;
        const int chunk = ld_c ^ ((row >> 1) & 7);
        b_goff[i] = (uint32_t)min(row, N - 1 - n0) * (uint32_t)K + chunk * 16;
    }
    // scale request i of a wavefront: scale dword i % SDW of the K step, for 64-row group a_grp(i) / b_grp(i)
    constexpr int SDW = Cfg::SDW;
    auto a_grp = [&](int i) __attribute__((always_inline)) { return (wave + (i / SDW) * Cfg::WAVES) % (Cfg::BM / 64); };
    auto b_grp = [&](int i) __attribute__((always_inline)) { return (wave + (i / SDW) * Cfg::WAVES) % (Cfg::BN / 64); };
#pragma unroll
    for (int i = 0; i < Cfg::SA_LOADS; ++i)
        as_goff[i] = (uint32_t)min(a_grp(i) * 64 + lane, M - 1 - m0) * (uint32_t)nkb;
#pragma unroll
    for (int i = 0; i < Cfg::SB_LOADS; ++i)
        bs_goff[i] = (uint32_t)min(b_grp(i) * 64 + lane, N - 1 - n0) * (uint32_t)nkb;
    const uint8_t *a_tile = a_q + (int64_t)m0 * K + k0, *b_tile = b_q + (int64_t)n0 * K + k0;
    const uint8_t *as_tile = a_s + (int64_t)m0 * nkb + k0 / Cfg::SBLK, *bs_tile = b_s + (int64_t)n0 * nkb + k0 / Cfg::SBLK;
    // Tiled scales: the 64 dwords of a (64-row group, K step) are contiguous, so the instruction that
    // reads one cache line per lane from row-major scales reads 256 consecutive bytes here. A ragged
    // last tile re-reads the last valid group: its rows are never stored.
    const uint8_t *as_grp[Cfg::SA_LOADS + 1], *bs_grp[Cfg::SB_LOADS + 1];
    if constexpr (TILED) {
#pragma unroll
        for (int i = 0; i < Cfg::SA_LOADS; ++i)
            as_grp[i] = a_s + ((int64_t)min(m0 / 64 + a_grp(i), (M + 63) / 64 - 1) * KT_row + k0 / BK) * (256 * SDW);
#pragma unroll
        for (int i = 0; i < Cfg::SB_LOADS; ++i)
            bs_grp[i] = b_s + ((int64_t)min(n0 / 64 + b_grp(i), (N + 63) / 64 - 1) * KT_row + k0 / BK) * (256 * SDW);
    }
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);

    // DMA slot t (compile-time after unrolling) of the A / B loads of K step kt into buffer buf
    auto issue_a = [&](int t, int kt, int buf) __attribute__((always_inline)) {
        if (t < Cfg::A_LOADS) {
            dma_load<16>(a_tile + (int64_t)kt * BK, a_goff[t],
                         lds_base + Cfg::A_OFF + buf * Cfg::A_BYTES + (wave * Cfg::A_LOADS + t) * 1024);
        } else if (t < Cfg::NA) {
            const int i = t - Cfg::A_LOADS;
            // every wavefront issues the same number of requests (the wait counts rely on it):
            // with fewer 64-row groups than wavefronts some groups are simply fetched twice
            const int dw = i % SDW;
            if constexpr (TILED)
                dma_load<4>(as_grp[i] + ((int64_t)kt * SDW + dw) * 256, lane * 4,
                            lds_base + Cfg::SA_OFF + buf * Cfg::SA_BYTES + dw * Cfg::BM * 4 + a_grp(i) * 256);
            else
                dma_load<4>(as_tile + (kt * SDW + dw) * 4, as_goff[i],
                            lds_base + Cfg::SA_OFF + buf * Cfg::SA_BYTES + dw * Cfg::BM * 4 + a_grp(i) * 256);
        }
    };
    auto issue_b = [&](int t, int kt, int buf) __attribute__((always_inline)) {
        if (t < Cfg::B_LOADS) {
            dma_load<16>(b_tile + (int64_t)kt * BK, b_goff[t],
                         lds_base + Cfg::B_OFF + buf * Cfg::B_BYTES + (wave * Cfg::B_LOADS + t) * 1024);
        } else if (t < Cfg::NB) {
            const int i = t - Cfg::B_LOADS;
            const int dw = i % SDW;
            if constexpr (TILED)
                dma_load<4>(bs_grp[i] + ((int64_t)kt * SDW + dw) * 256, lane * 4,
                            lds_base + Cfg::SB_OFF + buf * Cfg::SB_BYTES + dw * Cfg::BN * 4 + b_grp(i) * 256);
            else
                dma_load<4>(bs_tile + (kt * SDW + dw) * 4, bs_goff[i],
                            lds_base + Cfg::SB_OFF + buf * Cfg::SB_BYTES + dw * Cfg::BN * 4 + b_grp(i) * 256);
        }
    };

    // ---- fragment addresses (bytes inside an A or B buffer): row*128 + swizzled 16-byte chunk for
    // the two K halves a lane holds; tile i sits 16 rows = 2048 bytes further (the swizzle term
    // (row/2)%8 does not change with multiples of 16 rows). Scale byte: row*4 + K block.
    const int a_row = wm * Cfg::WM + r16, b_row = wn * Cfg::WN + r16;
    const int a_off0 = a_row * BK + ((g ^ ((a_row >> 1) & 7)) << 4), a_off1 = a_row * BK + (((4 + g) ^ ((a_row >> 1) & 7)) << 4);
    const int b_off0 = b_row * BK + ((g ^ ((b_row >> 1) & 7)) << 4), b_off1 = b_row * BK + (((4 + g) ^ ((b_row >> 1) & 7)) << 4);
    const int a_soff = a_row * 4 + g, b_soff = b_row * 4 + g;
    auto read_frag = [&](const uint8_t *base, int off0, int off1) __attribute__((always_inline)) {
        const v4i lo = *reinterpret_cast<const v4i *>(base + off0);
        const v4i hi = *reinterpret_cast<const v4i *>(base + off1);
        return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };

    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    v8i fa[TM];  // A fragments and scale bytes of the current step (refilled in place, see below)
    int sa[TM];

    // ---- one K step (buffers cur = kt & 1, nxt = the other one) ----------------------------------
    // State on entry: the A fragments and A scale bytes of step kt are in registers (fa, sa); B(kt)
    // is in LDS buffer cur; A(kt+1) is in flight towards (or already in) A buffer nxt.
    //   column 0      : MFMAs start at once (only the first B fragment has to arrive); the B tile of
    //                   step kt+1 is requested into B buffer nxt, one DMA instruction per MFMA;
    //   columns 1..-2 : B fragments stream through two register sets; the A tile of step kt+2 is
    //                   requested into A buffer cur (its fragments were pulled into registers during
    //                   the previous step), in the second half of each column, when the prefetch
    //                   read of the next B fragment has drained from the LDS queue;
    //   barrier M     : wait until only the requests of this step are outstanding, i.e. A(kt+1) has
    //                   landed for every wavefront;
    //   last column   : after MFMA (i, last) the registers of A fragment i are dead and are refilled
    //                   in place with fragment i of A(kt+1): the fragment reads of the next step are
    //                   spread over this column instead of bursting at its start;
    //   barrier E     : wait until B(kt+1) has landed (only this step's A requests may be pending).
    // So B is fetched one step ahead, A almost two, with 96 KB in flight against 64 KB in use.
    constexpr int A_LO = (TN - 2) * (TM - TM / 2) >= Cfg::NA ? TM / 2 : 0;  // first MFMA of a column that issues
    static_assert((TN - 2) * (TM - A_LO) >= Cfg::NA, "A requests fit into columns 1..TN-2");
    auto step = [&](int kt) __attribute__((always_inline)) {
        const int cur = kt & 1, nxt = cur ^ 1;
        // past the end of K the prefetches fetch the last step again into buffers nobody reads any
        // more: every step runs the same branch-free code and the wait counts stay valid
        const int kt1 = min(kt + 1, KT - 1), kt2 = min(kt + 2, KT - 1);
        const uint8_t *bbuf = lds + Cfg::B_OFF + cur * Cfg::B_BYTES, *sbbuf = lds + Cfg::SB_OFF + cur * Cfg::SB_BYTES;
        const uint8_t *anext = lds + Cfg::A_OFF + nxt * Cfg::A_BYTES, *sanext = lds + Cfg::SA_OFF + nxt * Cfg::SA_BYTES;
        // B fragments stream through NFB register sets, fetched NFB-1 columns ahead of their use
        constexpr int NFB = 3;
        v8i fb[NFB];
        int sb[NFB];
#pragma unroll
        for (int j = 0; j < NFB - 1 && j < TN; ++j) {
            fb[j] = read_frag(bbuf, b_off0 + j * 2048, b_off1 + j * 2048);
            sb[j] = read_scale<Cfg>(sbbuf, b_soff + j * 64, Cfg::BN);
        }
        MXFP8_PIN();
        int a_slot = 0;  // compile-time after unrolling
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (j + NFB - 1 < TN) {
                fb[(j + NFB - 1) % NFB] = read_frag(bbuf, b_off0 + (j + NFB - 1) * 2048, b_off1 + (j + NFB - 1) * 2048);
                sb[(j + NFB - 1) % NFB] = read_scale<Cfg>(sbbuf, b_soff + (j + NFB - 1) * 64, Cfg::BN);
            }
            if (j == TN - 1) {
                MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB);  // all but this step's requests: A(kt+1) is in LDS
                __syncthreads();
            }
            MXFP8_PIN();
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                acc[i][j] = mma_step<Cfg>(fb[j % NFB], fa[i], acc[i][j], sb[j % NFB], sa[i]);
                MXFP8_PIN();
                if (j == 0) {
                    issue_b(i, kt1, nxt);
                    if (i + TM < Cfg::NB)
                        issue_b(i + TM, kt1, nxt);
                } else if (j < TN - 1 && i >= A_LO) {
                    if (a_slot < Cfg::NA)
                        issue_a(a_slot, kt2, cur);
                    ++a_slot;
                }
                if (j == TN - 1) {
                    fa[i] = read_frag(anext, a_off0 + i * 2048, a_off1 + i * 2048);
                    sa[i] = read_scale<Cfg>(sanext, a_soff + i * 64, Cfg::BM);
                }
                MXFP8_PIN();
            }
        }
        MXFP8_WAIT_VMCNT(Cfg::NA);  // everything older than this step's A requests: B(kt+1) is in LDS
        __syncthreads();
    };

    if (KT > 0) {
#pragma unroll
        for (int t = 0; t < Cfg::NA; ++t)
            issue_a(t, 0, 0);
#pragma unroll
        for (int t = 0; t < Cfg::NB; ++t)
            issue_b(t, 0, 0);
#pragma unroll
        for (int t = 0; t < Cfg::NA; ++t)
            issue_a(t, min(1, KT - 1), 1);
        MXFP8_WAIT_VMCNT(0);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            fa[i] = read_frag(lds + Cfg::A_OFF, a_off0 + i * 2048, a_off1 + i * 2048);
            sa[i] = read_scale<Cfg>(lds + Cfg::SA_OFF, a_soff + i * 64, Cfg::BM);
        }
        __syncthreads();  // A buffer 0 is refilled by the requests of step 0 from here on
    }
    for (int kt = 0; kt < KT; ++kt)
        step(kt);
    MXFP8_WAIT_VMCNT(0);  // drain the redundant tail prefetches before the LDS allocation is released

    // ---- epilogue: lane (r16, g) of tile (i, j) holds C[m0w + 16i + r16][n0w + 16j + 4g + 0..3]
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * Cfg::WM + i * 16 + r16;
        if (m >= M)
            continue;
        uint8_t *crow = c + (int64_t)m * ldc_bytes;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + wn * Cfg::WN + j * 16 + 4 * g;
            const v4f v = acc[i][j];
            if (vec_store && n + 3 < N) {
                if constexpr (OUT_BF16) {
                    v2bf p0 = {(__bf16)v[0], (__bf16)v[1]}, p1 = {(__bf16)v[2], (__bf16)v[3]};
                    *reinterpret_cast<uint2 *>(crow + (int64_t)n * 2) =
                        make_uint2(__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1));
                } else {
                    *reinterpret_cast<float4 *>(crow + (int64_t)n * 4) = make_float4(v[0], v[1], v[2], v[3]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) {
                        if constexpr (OUT_BF16)
                            *reinterpret_cast<__bf16 *>(crow + (int64_t)(n + e) * 2) = (__bf16)v[e];
                        else
                            *reinterpret_cast<float *>(crow + (int64_t)(n + e) * 4) = v[e];
                    }
            }
        }
    }
}

// ---- persistent variant --------------------------------------------------------------------------
// One workgroup per compute unit walks over several output tiles and keeps the K pipeline running
// across tile boundaries: the prefetches of the last two K steps of a tile, which the kernel above
// spends on re-reading the last step, fetch the first steps of the workgroup's next tile instead, so
// only the first tile of a workgroup has a prologue, and the epilogue stores of a tile drain while
// the operands of the next one are already in flight. Needs M >= BM, N >= BN, K >= 2 steps and vector-storable C.
// The last tile of a ragged row or column of tiles is moved back so that it ends with the operand: its first rows or
// columns are computed twice, by the same instructions, and stored by their own tile only. So the DMA offsets inside a
// tile are the same for every tile and no request needs a clamp.
// Wait counts: the epilogue's stores also count in vmcnt. Loads complete in order among themselves,
// so "at most n operations outstanding" still implies that all but the last n loads have landed,
// whatever the stores do; the immediates of the K step stay valid (they can only wait longer).
// FUSE_Q (BF16 output only; bit 0 = row-wise copy, bit 1 = column-wise copy): the epilogue also emits MXFP8 copies of the
// BF16 output tile (Section 2: the output is re-quantized when the next layer needs it in MX format), scales in the same
// layout as the inputs: cq [M x N], cs = scales of C as an [M x N] operand; cqT [N x M], csT = scales of C^T.
//   row-wise alone: straight from the accumulators; a 32-column block lies in two adjacent MFMA tiles of one row, 8 values
//     in each of the 4 lanes that share the row. ([8192 x 14336 x 4096]: 389 us, 417 us by way of the tile read back.)
//   with a column-wise copy: as soon as the tile is stored, the workgroup reads it back (from the L2 it was just written
//     to) in 128x128 pieces and converts those like the quantizer does. Straight from the accumulators this needs the amax
//     and the transposed bytes of values that lie spread over 16 lanes: it spilled 316 bytes per work-item and took 42 us
//     per 256x256 tile ([4096 x 14336 x 4096], both copies: 337 us, 259 us this way).
#ifndef MXFP8_GEMM_SCHED
#define MXFP8_GEMM_SCHED 242  // B requests behind every 2nd MFMA, a gap of 2, A requests behind every 4th
#endif
struct KExpert {
    int steps, first, expert;  // K steps, the first of them, whose they are
};
constexpr int kMostKExperts = 128;  // that the K-grouped form sorts
// Who computes which tile of the K-grouped form: rounds over the workgroups, every other one backwards; the first `busy` workgroups
// have no tile in rounds 1 .. skipped.
struct KShares {
    int busy, skipped;
    // number of the tile that workgroup b computes as its `index`th (from 0 on; growing with it)
    __device__ __forceinline__ int tile(int b, int index) const
    {
        const int round = index > 0 && b < busy ? index + skipped : index;
        const int out = round > 0 && round <= skipped ? busy : 0, width = (int)gridDim.x - out, place = b - out;
        return round * (int)gridDim.x - min(max(round - 1, 0), skipped) * busy + (round & 1 ? width - 1 - place : place);
    }
};
// GROUPED (Appendix A.4, mixture-of-experts layers): the rows of A are tokens sorted by expert, rows
// [group_ends[e-1], group_ends[e]) belong to expert e, whose B operand starts b_group_bytes (scales:
// bs_group_bytes) after the previous expert's. group_ends lives in DEVICE memory (routing happens on the
// GPU), so the host cannot count the tiles: every workgroup sums them up itself, walks over its share and
// finds the expert of a tile by scanning the ends (wavefront-uniform scalar code, a few hundred cycles per
// 100 k-cycle tile). An expert's last tile may be partial: its surplus rows are computed from whatever
// rows follow (the next expert's, or re-reads of the last row of A) and not stored. N stays a multiple of
// the tile. Ends are clamped to [previous end, M], so bad ends cannot send a load out of A.
// RAGGED: M or N is no multiple of the tile (a kernel of its own, so that whole tiles carry no masks: 1 % of their time).
// KGROUPED (weight gradient of a mixture-of-experts layer, see the kernel above): the tiles of all experts that have whole K
// steps, each with a K range of its own; down to one step, so that the A requests, two steps ahead, can reach into the tile after
// the next one. Experts without a step get zeros, rows spread over the workgroups. What bounds it: the FP32 output (8 experts x
// [5632 x 2048] from 8192 tokens: 369 MB, 60 us of writing) and 9 steps of 1.5 us per tile, one after the other where all units
// store at the same time.
// A workgroup's share is fixed before it starts, so it is shared out by what tiles take: the experts with the most steps first, every
// other round over the workgroups backwards, and where one expert has most of the steps its workgroups sit out some rounds
// (KShares). One after the other in the experts' order, loads that repeat with the rounds gave all long tiles to the same
// workgroups. In us, one tile per workgroup | in the experts' order | this way (tiled scales, FP32 out): [2048 x 2048], experts of
// 49,5,5,5,49,5,5,5 steps 97.8 | 136.5 | 92.8; [4096 x 2048], 64 experts of 31 and 1 by turns 1521 | 2100 | 1266; [2816 x 2048], 64
// experts, one with 256 of 508 steps 885 | 1074 | 867, and eight each 679 | 626 | 552; [5632 x 2048], eight of eight steps 154 | 135 | 132.
// Not so where the steps fall off like 1/i: [2048 x 2048], 16 experts of 128 steps 119 | 144 | 125.
template <class Cfg, bool OUT_BF16, bool TILED, bool SPREAD, int FUSE_Q = 0, int SCHED = MXFP8_GEMM_SCHED, bool GROUPED = false, bool RAGGED = false,
          bool KGROUPED = false>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_persistent_kernel(
    const uint8_t *__restrict__ a_q, const uint8_t *__restrict__ a_s, const uint8_t *__restrict__ b_q,
    const uint8_t *__restrict__ b_s, int M, int N, int K, uint8_t *__restrict__ c, int64_t ldc_bytes,
    int tiles_m, int tiles_n, uint8_t *__restrict__ cq, uint8_t *__restrict__ cs, uint8_t *__restrict__ cqT,
    uint8_t *__restrict__ csT, GemmGroups groups, GemmTail tail)
{
    static_assert(!(GROUPED || KGROUPED) || (FUSE_Q == 0 && Cfg::ALL_E4M3), "grouped products: MXFP8-E4M3 operands, plain epilogue");
    static_assert(!GROUPED || (!RAGGED && !KGROUPED), "rows and K steps are not grouped at once");
    static_assert(!FUSE_Q || (OUT_BF16 && Cfg::BM % kTile == 0 && Cfg::BN % kTile == 0 && Cfg::THREADS == kQuantThreads), "fused output quantization");
    constexpr bool Q_ROW_ONLY = FUSE_Q == 1;
    static_assert(!Q_ROW_ONLY || Cfg::TN == 8 || Cfg::TN == 4, "the scale bytes of a row are a dword or a halfword");
    static_assert(!FUSE_Q || Cfg::WAVES * kStageBytes >= kTile * kTile + 2 * kTile * 4, "the converted tile fits the staging areas");
    static_assert(!Cfg::SCALED || (Cfg::SA_LOADS == Cfg::SDW && Cfg::SB_LOADS == Cfg::SDW), "one scale request per wavefront, operand and scale dword");
    static_assert(Cfg::ALL_E4M3 || FUSE_Q == 0, "output quantization belongs to the MXFP8-E4M3 product");
    MXFP8_DYNAMIC_LDS(lds);
    constexpr int TM = Cfg::TM, TN = Cfg::TN;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;
    const int r16 = lane & 15, g = lane >> 4;
    constexpr int SDW = Cfg::SDW;
    const int nkb = K / Cfg::SBLK;
    const int KT = K / BK;
    int ntiles = tiles_m * tiles_n;
    if constexpr (GROUPED)
        ntiles = grouped_tiles<Cfg::BM>(groups, M, tiles_n);
    [[maybe_unused]] KExpert *const by_steps = reinterpret_cast<KExpert *>(lds + Cfg::LDS_BYTES_PERSISTENT);
    [[maybe_unused]] KShares shares = {0, 0};
    if constexpr (KGROUPED) {
        static_assert(Cfg::THREADS == 2 * kMostKExperts && kMostKExperts == 2 * 64, "two work-items per expert, two experts per lane");
        const int per_expert = ntiles, pieces = N * (OUT_BF16 ? 2 : 4) / 16;
        // Lane l of every wavefront has the experts 2 l and 2 l + 1; an end is the largest one up to there, at most K. Reading one
        // expert after the other took 60 ns each, before a tile's first request. In us, one tile per workgroup | one expert after the
        // other | this way: [512 x 512], 64 experts of 2 and of 6 steps (tiled scales, BF16 out) 22.5 | 26.3 | 18.3 and 31.8 | 35.0 |
        // 27.2; [1024 x 1024], 16 experts of 6 steps (row-major scales, FP32 out) 29.7 | 31.6 | 29.0.
        auto end_of = [&](int e) { return e < groups.count ? min(max(groups.ends[e], 0), K) : 0; };
        int end0 = end_of(2 * lane), end1 = end_of(2 * lane + 1), top = max(end0, end1);
        for (int d = 1; d < 64; d *= 2)
            top = max(top, __shfl(top, max(lane - d, 0), 64));
        const int left = __shfl(top, max(lane - 1, 0), 64), before = lane > 0 ? left : 0;
        end0 = max(end0, before);
        end1 = max(end1, end0);
        const int first0 = before / BK, first1 = end0 / BK, steps0 = first1 - first0, steps1 = end1 / BK - first1;
        const int all = __builtin_amdgcn_readfirstlane(__shfl(top, 63, 64)) / BK;  // steps of all experts
        const uint64_t has0 = __ballot(steps0 > 0), has1 = __ballot(steps1 > 0);
        const int active = __popcll(has0) + __popcll(has1);
        ntiles = active * per_expert;
        // Zeros: where every tile has a workgroup, by those that are left over, else by all of them.
        const int writers = per_expert * groups.count <= (int)gridDim.x ? (int)gridDim.x - ntiles : (int)gridDim.x;
        const int writer = (int)blockIdx.x - ((int)gridDim.x - writers);
        if (active < groups.count && writer >= 0)
            for (int e = 0; e < groups.count; ++e)
                if (!(((e & 1) ? has1 : has0) >> (e >> 1) & 1))
                    for (int m = writer; m < M; m += writers)
                        for (int i = tid; i < pieces; i += Cfg::THREADS)
                            *reinterpret_cast<uint4 *>(c + ((int64_t)e * M + m) * ldc_bytes + (int64_t)i * 16) = make_uint4(0, 0, 0, 0);
        int32_t *const scratch = reinterpret_cast<int32_t *>(lds);
        const bool one_round = ntiles <= (int)gridDim.x;
        if (one_round) {  // a workgroup has one tile at most: in the experts' order
            if (wave == 0) {
                const uint64_t below = ((uint64_t)1 << lane) - 1;
                int rank = __popcll(has0 & below) + __popcll(has1 & below);
                if (steps0 > 0)
                    by_steps[rank++] = {steps0, first0, 2 * lane};
                if (steps1 > 0)
                    by_steps[rank] = {steps1, first1, 2 * lane + 1};
            }
        } else {  // in the order of their steps, most of them first
            uint32_t *const keys = reinterpret_cast<uint32_t *>(lds);  // of all kMostKExperts; no two are the same
            if (wave == 0) {
                keys[2 * lane] = (uint32_t)steps0 * kMostKExperts + (kMostKExperts - 1 - 2 * lane);
                keys[2 * lane + 1] = (uint32_t)steps1 * kMostKExperts + (kMostKExperts - 2 - 2 * lane);
                scratch[kMostKExperts + 2 * lane] = first0;
                scratch[kMostKExperts + 2 * lane + 1] = first1;
            }
            __syncthreads();
            const int expert = tid >> 1;
            const uint32_t key = keys[expert];
            int rank = 0;
            for (int e = 4 * (tid & 1); e < groups.count; e += 8) {
                const uint4 k = *reinterpret_cast<const uint4 *>(keys + e);
                rank += (k.x > key) + (k.y > key) + (k.z > key) + (k.w > key);
            }
            rank += __shfl_xor(rank, 1, 64);
            if ((tid & 1) == 0 && expert < groups.count)
                by_steps[rank] = {(int)(key / kMostKExperts), scratch[kMostKExperts + expert], expert};
        }
        __syncthreads();
        // Where one expert has far more steps than the others have on average, the workgroups with its tiles sit out the rounds
        // in which the others catch up, if that makes the longest share shorter (in steps; an estimate).
        constexpr int STORE = OUT_BF16 ? 4 : 8;  // what a tile takes besides its K loop
        const int most = one_round ? 0 : __builtin_amdgcn_readfirstlane(by_steps[0].steps);
        const int others = all - most + STORE * (active - 1);
        const int rounds = !one_round && per_expert < (int)gridDim.x ? (most + STORE) * (active - 1) / others - 1 : 0;
        if (rounds > 0) {
            int longest[2] = {0, 0};  // without and with
            for (int b = tid; b < (int)gridDim.x; b += Cfg::THREADS)
                for (int with = 0; with < 2; ++with) {
                    const KShares how = {with ? per_expert : 0, with ? rounds : 0};
                    int share = 0;
                    for (int i = 0, u; (u = how.tile(b, i)) < ntiles; ++i)
                        share += by_steps[u / per_expert].steps + STORE;
                    longest[with] = max(longest[with], share);
                }
            for (int with = 0; with < 2; ++with) {
                for (int mask = 32; mask > 0; mask >>= 1)
                    longest[with] = max(longest[with], __shfl_xor(longest[with], mask, 64));
                scratch[2 * wave + with] = longest[with];
            }
            __syncthreads();
            for (int w = 0; w < Cfg::WAVES; ++w)
                for (int with = 0; with < 2; ++with)
                    longest[with] = max(longest[with], scratch[2 * w + with]);
            if (__builtin_amdgcn_readfirstlane(longest[1]) < __builtin_amdgcn_readfirstlane(longest[0]))
                shares = {per_expert, rounds};
            __syncthreads();
        }
    }
    const int stride = gridDim.x;
    // >= 1 when the host knows the number of tiles (the grid has at most that many workgroups)
    int my_tiles = (tail.first(ntiles) - (int)blockIdx.x + stride - 1) / stride;
    if constexpr (KGROUPED)
        for (my_tiles = 0; shares.tile((int)blockIdx.x, my_tiles) < ntiles;)
            ++my_tiles;
    if ((GROUPED || KGROUPED) && my_tiles <= 0)
        return;  // the whole workgroup, before any barrier

    // ---- DMA offsets inside an operand tile (see the kernel above); the same for every tile.
    const int ld_r = lane >> 3, ld_c = lane & 7;
    uint32_t a_goff[Cfg::A_LOADS], b_goff[Cfg::B_LOADS];
#pragma unroll
    for (int i = 0; i < Cfg::A_LOADS; ++i) {
        const int row = (wave * Cfg::A_LOADS + i) * 8 + ld_r;
        a_goff[i] = (uint32_t)row * (uint32_t)K + (ld_c ^ ((row >> 1) & 7)) * 16;
    }
#pragma unroll
    for (int i = 0; i < Cfg::B_LOADS; ++i) {
        const int row = (wave * Cfg::B_LOADS + i) * 8 + ld_r;
        b_goff[i] = (uint32_t)row * (uint32_t)K + (ld_c ^ ((row >> 1) & 7)) * 16;
    }
    // 64-row groups of the A and the B tile whose scale dwords this wavefront fetches
    const int a_grp = wave % (Cfg::BM / 64), b_grp = wave % (Cfg::BN / 64);
    const int s_step = (TILED ? 256 : 4) * SDW;  // bytes from the scale dwords of one K step to the next
    constexpr int s_dword = TILED ? 256 : 4;     // ... and from one scale dword of a K step to its next one
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);

    // operand pointers of a tile at K step 0 (wavefront-uniform). What only the K-grouped form needs is no member of the others.
    struct Nothing {};
    struct Range {
        int steps;   // K steps of the tile's expert
        uint8_t *c;  // output of the tile's expert
    };
    struct Tile : std::conditional_t<KGROUPED, Range, Nothing> {
        const uint8_t *a, *b, *as, *bs;
        int m0, n0;
        uint32_t as_off, bs_off;  // this lane's offset from as / bs
        int row_lo, col_lo;  // rows and columns of the tile before these are another tile's (not stored)
        int rows;  // GROUPED: rows of the tile that belong to its expert (stored)
        int lim;   // GROUPED: last row of the tile, counted from m0, that may be read from A
    };
    // Scale requests of the 64 operand rows from `first` on: base and this lane's offset. Tiled scales keep 64 rows
    // together, but a tile that was moved back may begin between two such groups.
    auto scale_rows = [&](const uint8_t *s, int first, const uint8_t *&base, uint32_t &off) __attribute__((always_inline)) {
        if constexpr (TILED) {
            base = s + (int64_t)(first >> 6) * KT * (256 * SDW);
            off = lane * 4;
            if constexpr (RAGGED) {
                const int row = first + lane;
                off = (uint32_t)((row >> 6) - (first >> 6)) * (uint32_t)(KT * 256 * SDW) + (row & 63) * 4;
            }
        } else {
            base = s + (int64_t)first * nkb;
            off = (uint32_t)lane * (uint32_t)nkb;
        }
    };
    auto tile_at = [&](int index) __attribute__((always_inline)) {
        int tm, tn;
        Tile t;
        const uint8_t *bq = b_q, *bsc = b_s;
        [[maybe_unused]] int first_step = 0;  // KGROUPED: where the expert's K range starts
        if constexpr (GROUPED) {
            // The workgroups that run side by side have consecutive ids: they work on the same expert (all
            // XCDs then stream the same B operand), and inside the expert's tiles the XCD-aware order applies.
            const GroupTile at = grouped_tile<Cfg::BM>(groups, M, tiles_n, (int)blockIdx.x + index * stride);
            tm = at.tm;
            tn = at.tn;
            t.m0 = at.begin + at.tm * Cfg::BM;
            t.rows = min(Cfg::BM, at.end - t.m0);
            t.lim = M - 1 - t.m0;
            bq += at.expert * groups.b_group_bytes;
            bsc += at.expert * groups.bs_group_bytes;
        } else {
            int u = (int)blockIdx.x + index * stride, count = ntiles;
            if constexpr (KGROUPED) {
                u = shares.tile((int)blockIdx.x, index);
                count = tiles_m * tiles_n;
                const int rank = u / count;
                u -= rank * count;
                t.steps = __builtin_amdgcn_readfirstlane(by_steps[rank].steps);
                first_step = __builtin_amdgcn_readfirstlane(by_steps[rank].first);
                t.c = c + (int64_t)__builtin_amdgcn_readfirstlane(by_steps[rank].expert) * M * ldc_bytes;
            }
            tile_of_block(u, count, tiles_m, tiles_n, tm, tn);
            // the last tile of a ragged row or column of tiles ends with the operand
            t.m0 = RAGGED ? min(tm * Cfg::BM, M - Cfg::BM) : tm * Cfg::BM;
            t.rows = Cfg::BM;
            t.lim = Cfg::BM;
        }
        t.n0 = RAGGED ? min(tn * Cfg::BN, N - Cfg::BN) : tn * Cfg::BN;
        t.row_lo = RAGGED ? tm * Cfg::BM - t.m0 : 0;
        t.col_lo = tn * Cfg::BN - t.n0;
        t.a = a_q + (int64_t)t.m0 * K;
        t.b = bq + (int64_t)t.n0 * K;
        if constexpr (GROUPED && TILED) {
            // group starts are multiples of 64 rows; 64-row groups past the end of A re-read the last one
            t.as = a_s + (int64_t)min(t.m0 / 64 + a_grp, (M + 63) / 64 - 1) * KT * (256 * SDW);
            t.as_off = lane * 4;
        } else if constexpr (GROUPED) {
            // from the tile's first row on: a request past the end of A takes rows off this offset (see issue_a)
            t.as = a_s + (int64_t)t.m0 * nkb;
            t.as_off = (uint32_t)(a_grp * 64 + lane) * (uint32_t)nkb;
        } else {
            scale_rows(a_s, t.m0 + a_grp * 64, t.as, t.as_off);
        }
        scale_rows(bsc, t.n0 + b_grp * 64, t.bs, t.bs_off);
        if constexpr (KGROUPED) {
            t.a += first_step * BK;
            t.b += first_step * BK;
            t.as += first_step * s_step;
            t.bs += first_step * s_step;
        }
        return t;
    };

    // DMA slot t of the A / B requests of one K step, from the step's source pointers into buffer buf.
    // GROUPED: rows of the A tile past `lim` (the end of A) re-read row lim.
    const int row0 = wave * Cfg::A_LOADS * 8 + ld_r;  // this lane's row in DMA slot 0
    auto issue_a = [&](int t, const uint8_t *src, const uint8_t *ssrc, uint32_t soff, int buf, int lim) __attribute__((always_inline)) {
        if (t < Cfg::A_LOADS) {
            uint32_t off = a_goff[t];
            if constexpr (GROUPED)
                off -= (uint32_t)max(row0 + 8 * t - lim, 0) * (uint32_t)K;
            dma_load<16>(src, off, lds_base + Cfg::A_OFF + buf * Cfg::A_BYTES + (wave * Cfg::A_LOADS + t) * 1024);
        } else if (t < Cfg::NA) {
            uint32_t off = soff;
            if constexpr (GROUPED && !TILED)
                off -= (uint32_t)max(a_grp * 64 + lane - lim, 0) * (uint32_t)nkb;
            const int dw = t - Cfg::A_LOADS;
            dma_load<4>(ssrc + dw * s_dword, off, lds_base + Cfg::SA_OFF + buf * Cfg::SA_BYTES + dw * Cfg::BM * 4 + a_grp * 256);
        }
    };
    auto issue_b = [&](int t, const uint8_t *src, const uint8_t *ssrc, uint32_t soff, int buf) __attribute__((always_inline)) {
        if (t < Cfg::B_LOADS)
            dma_load<16>(src, b_goff[t], lds_base + Cfg::B_OFF + buf * Cfg::B_BYTES + (wave * Cfg::B_LOADS + t) * 1024);
        else if (t < Cfg::NB)
            dma_load<4>(ssrc + (t - Cfg::B_LOADS) * s_dword, soff,
                        lds_base + Cfg::SB_OFF + buf * Cfg::SB_BYTES + (t - Cfg::B_LOADS) * Cfg::BN * 4 + b_grp * 256);
    };

    const int a_row = wm * Cfg::WM + r16, b_row = wn * Cfg::WN + r16;
    const int a_off0 = a_row * BK + ((g ^ ((a_row >> 1) & 7)) << 4), a_off1 = a_row * BK + (((4 + g) ^ ((a_row >> 1) & 7)) << 4);
    const int b_off0 = b_row * BK + ((g ^ ((b_row >> 1) & 7)) << 4), b_off1 = b_row * BK + (((4 + g) ^ ((b_row >> 1) & 7)) << 4);
    const int a_soff = a_row * 4 + g, b_soff = b_row * 4 + g;
    auto read_frag = [&](const uint8_t *base, int off0, int off1) __attribute__((always_inline)) {
        const v4i lo = *reinterpret_cast<const v4i *>(base + off0);
        const v4i hi = *reinterpret_cast<const v4i *>(base + off1);
        return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };

    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    v8i fa[TM];
    int sa[TM];

    // One K step, same schedule as in the kernel above; the requests go to the sources handed in:
    // (b_src, bs_src) = B tile and scales of the workgroup's NEXT step, (a_src, as_src) = A tile and
    // scales of the step after that, either of which may belong to the next output tile.
    constexpr int A_LO = (TN - 2) * (TM - TM / 2) >= Cfg::NA ? TM / 2 : 0;
    static_assert((TN - 2) * (TM - A_LO) >= Cfg::NA, "A requests fit into columns 1..TN-2");
    uint32_t as_off = 0, bs_off = 0;  // the lane's scale offsets of the tiles that as_src and bs_src belong to
    auto step = [&](int cur, const uint8_t *b_src, const uint8_t *bs_src, const uint8_t *a_src,
                    const uint8_t *as_src, int a_lim) __attribute__((always_inline)) {
        const int nxt = cur ^ 1;
        const uint8_t *bbuf = lds + Cfg::B_OFF + cur * Cfg::B_BYTES, *sbbuf = lds + Cfg::SB_OFF + cur * Cfg::SB_BYTES;
        const uint8_t *anext = lds + Cfg::A_OFF + nxt * Cfg::A_BYTES, *sanext = lds + Cfg::SA_OFF + nxt * Cfg::SA_BYTES;
        constexpr int NFB = 3;  // B fragment register sets, read NFB-1 columns ahead
        v8i fb[NFB];
        int sb[NFB];
#pragma unroll
        for (int j = 0; j < NFB - 1 && j < TN; ++j) {
            fb[j] = read_frag(bbuf, b_off0 + j * 2048, b_off1 + j * 2048);
            sb[j] = read_scale<Cfg>(sbbuf, b_soff + j * 64, Cfg::BN);
        }
        MXFP8_PIN();
        int a_slot = 0;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (j + NFB - 1 < TN) {
                fb[(j + NFB - 1) % NFB] = read_frag(bbuf, b_off0 + (j + NFB - 1) * 2048, b_off1 + (j + NFB - 1) * 2048);
                sb[(j + NFB - 1) % NFB] = read_scale<Cfg>(sbbuf, b_soff + (j + NFB - 1) * 64, Cfg::BN);
            }
            if (j == TN - 1) {
                MXFP8_WAIT_VMCNT(Cfg::NA + Cfg::NB);
                MXFP8_BARRIER();
            }
            MXFP8_PIN();
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                acc[i][j] = mma_step<Cfg>(fb[j % NFB], fa[i], acc[i][j], sb[j % NFB], sa[i]);
                MXFP8_PIN();
                if constexpr (SPREAD) {
                    // SCHED = 100 * gap + 10 * A spacing + B spacing (in MFMAs)
                    constexpr int B_EVERY = SCHED % 10, A_EVERY = SCHED / 10 % 10, GAP = SCHED / 100;
                    constexpr int A_FIRST = B_EVERY * Cfg::NB + GAP;  // MFMA after which the first A request goes out
                    static_assert(A_FIRST + A_EVERY * (Cfg::NA - 1) < (TN - 1) * TM, "all requests before the last column");
                    const int m = j * TM + i;  // compile-time after unrolling
                    if (m % B_EVERY == 0 && m / B_EVERY < Cfg::NB)
                        issue_b(m / B_EVERY, b_src, bs_src, bs_off, nxt);
                    else if (m >= A_FIRST && (m - A_FIRST) % A_EVERY == 0 && (m - A_FIRST) / A_EVERY < Cfg::NA)
                        issue_a((m - A_FIRST) / A_EVERY, a_src, as_src, as_off, cur, a_lim);
                } else if (j == 0) {
                    issue_b(i, b_src, bs_src, bs_off, nxt);
                    if (i + TM < Cfg::NB)
                        issue_b(i + TM, b_src, bs_src, bs_off, nxt);
                } else if (j < TN - 1 && i >= A_LO) {
                    if (a_slot < Cfg::NA)
                        issue_a(a_slot, a_src, as_src, as_off, cur, a_lim);
                    ++a_slot;
                }
                if (j == TN - 1) {
                    fa[i] = read_frag(anext, a_off0 + i * 2048, a_off1 + i * 2048);
                    sa[i] = read_scale<Cfg>(sanext, a_soff + i * 64, Cfg::BM);
                }
                MXFP8_PIN();
            }
        }
        // end of the step: B(k+1) has landed; B buffer cur and A buffer nxt go back to the DMA, so this
        // wavefront's refill reads of A buffer nxt must have returned before anybody passes the barrier
        MXFP8_WAIT_VMCNT_AND_LDS(Cfg::NA);
        MXFP8_BARRIER();
    };

    Tile cur_tile = tile_at(0);
    // KGROUPED: the tile after the next one; past the last tile, that one again
    std::conditional_t<KGROUPED, Tile, Nothing> after_next;
    // prologue of the workgroup's first tile: A(0), B(0) into buffers 0, A(1) into A buffer 1
    const uint8_t *a_second = cur_tile.a + BK, *as_second = cur_tile.as + s_step;
    uint32_t as_off_second = cur_tile.as_off;
    if constexpr (KGROUPED) {
        after_next = my_tiles > 1 ? tile_at(1) : cur_tile;
        if (cur_tile.steps == 1) {
            a_second = after_next.a;
            as_second = after_next.as;
            as_off_second = after_next.as_off;
        }
    }
#pragma unroll
    for (int t = 0; t < Cfg::NA; ++t)
        issue_a(t, cur_tile.a, cur_tile.as, cur_tile.as_off, 0, cur_tile.lim);
#pragma unroll
    for (int t = 0; t < Cfg::NB; ++t)
        issue_b(t, cur_tile.b, cur_tile.bs, cur_tile.bs_off, 0);
#pragma unroll
    for (int t = 0; t < Cfg::NA; ++t)
        issue_a(t, a_second, as_second, as_off_second, 1, cur_tile.lim);
    MXFP8_WAIT_VMCNT(0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        fa[i] = read_frag(lds + Cfg::A_OFF, a_off0 + i * 2048, a_off1 + i * 2048);
        sa[i] = read_scale<Cfg>(lds + Cfg::SA_OFF, a_soff + i * 64, Cfg::BM);
    }
    __syncthreads();

    int par = 0;  // LDS buffer parity of the workgroup's running step count
    for (int ti = 0; ti < my_tiles; ++ti) {
        const bool has_next = ti + 1 < my_tiles;
        auto following = [&]() __attribute__((always_inline)) {
            if constexpr (KGROUPED)
                return after_next;
            else
                return has_next ? tile_at(ti + 1) : cur_tile;
        };
        const Tile next_tile = following();
        int steps = KT;
        if constexpr (KGROUPED) {
            after_next = ti + 2 < my_tiles ? tile_at(ti + 2) : next_tile;
            steps = cur_tile.steps;
        }
        for (int kt = 0; kt < steps; ++kt) {
            // source of the step after this one (B) and of the one after that (A): this tile, else the
            // first steps of the next tile, else (last tile) this tile's last step once more
            const uint8_t *b_src, *bs_src, *a_src, *as_src;
            int a_lim = cur_tile.lim;
            if constexpr (KGROUPED) {
                // step kt + 1 of this tile, or the next tile's first one (past the last tile its last step once more)
                const bool b_here = kt + 1 < steps || !has_next;
                const int b_step = b_here ? min(kt + 1, steps - 1) : 0;
                b_src = (b_here ? cur_tile.b : next_tile.b) + (int64_t)b_step * BK;
                bs_src = (b_here ? cur_tile.bs : next_tile.bs) + (int64_t)b_step * s_step;
                bs_off = b_here ? cur_tile.bs_off : next_tile.bs_off;
                // step kt + 2: this tile's, one of the next tile's first two, or, where that has one step only, the first
                // of the tile after it (after_next is the next tile itself where there is none)
                const bool a_here = kt + 2 < steps || !has_next;
                const bool a_next = kt + 2 - steps < next_tile.steps;
                const int a_step = a_here ? min(kt + 2, steps - 1) : a_next ? kt + 2 - steps : 0;
                a_src = (a_here ? cur_tile.a : a_next ? next_tile.a : after_next.a) + (int64_t)a_step * BK;
                as_src = (a_here ? cur_tile.as : a_next ? next_tile.as : after_next.as) + (int64_t)a_step * s_step;
                as_off = a_here ? cur_tile.as_off : a_next ? next_tile.as_off : after_next.as_off;
            } else {
                as_off = kt + 2 < KT ? cur_tile.as_off : next_tile.as_off;
                bs_off = kt + 1 < KT ? cur_tile.bs_off : next_tile.bs_off;
                if (kt + 1 < KT) {
                    b_src = cur_tile.b + (int64_t)(kt + 1) * BK;
                    bs_src = cur_tile.bs + (int64_t)(kt + 1) * s_step;
                } else if (has_next) {
                    b_src = next_tile.b;
                    bs_src = next_tile.bs;
                } else {
                    b_src = cur_tile.b + (int64_t)(KT - 1) * BK;
                    bs_src = cur_tile.bs + (int64_t)(KT - 1) * s_step;
                }
                if (kt + 2 < KT) {
                    a_src = cur_tile.a + (int64_t)(kt + 2) * BK;
                    as_src = cur_tile.as + (int64_t)(kt + 2) * s_step;
                } else if (has_next) {
                    a_src = next_tile.a + (int64_t)(kt + 2 - KT) * BK;
                    as_src = next_tile.as + (int64_t)(kt + 2 - KT) * s_step;
                    a_lim = next_tile.lim;
                } else {
                    a_src = cur_tile.a + (int64_t)(KT - 1) * BK;
                    as_src = cur_tile.as + (int64_t)(KT - 1) * s_step;
                }
            }
            step(par, b_src, bs_src, a_src, as_src, a_lim);
            par ^= 1;
        }
        // ---- epilogue of this tile; the A requests of the next tile's second step are in flight.
        // Row groups (16 rows of the wavefront's part) are finished one after the other (pinned), each through
        // the wavefront's staging area, so that the converted values of only one row group are live at a
        // time next to the A fragments of the next tile.
        constexpr int ESZ = OUT_BF16 ? 2 : 4;
        uint8_t *ctile = c;
        if constexpr (KGROUPED)
            ctile = cur_tile.c;
        ctile += (int64_t)cur_tile.m0 * ldc_bytes + (int64_t)cur_tile.n0 * ESZ;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            uint8_t *crow = ctile + (int64_t)(i * 16) * ldc_bytes;
            // the values of this row group are still in accumulator registers at this point: keeps the
            // compiler from moving all 256 of them into ordinary registers at the top of the epilogue
#pragma unroll
            for (int j = 0; j < TN; ++j)
                MXFP8_KEEP_IN_ACC(acc[i][j]);
            if constexpr (Q_ROW_ONLY) {
                // BF16 rows and their MXFP8 copy both leave through the wavefront's staging area (see the plain
                // epilogue below for why): first the 16 BF16 rows, then, in the same area, the 16 byte rows.
                const int64_t m = cur_tile.m0 + wm * Cfg::WM + i * 16 + r16;        // this lane's row of C
                const int n_wave = cur_tile.n0 + wn * Cfg::WN;                       // first column of the wavefront
                constexpr int ROWB = Cfg::WN * 2, PITCH = ROWB + 32;                 // BF16 row and its staged pitch
                constexpr int QPITCH = Cfg::WN + 16;                                 // staged pitch of a byte row
                static_assert(16 * PITCH <= kStageBytes && (16 * ROWB) % 1024 == 0 && (16 * Cfg::WN) % 1024 == 0, "staging area");
                uint8_t *stage = lds + Cfg::LDS_BYTES + wave * kStageBytes;
                uint32_t scales = 0;                                                 // scale bytes of the row's blocks
                uint32_t q[TN];
#pragma unroll
                for (int blk = 0; blk < TN / 2; ++blk) {
                    uint32_t h[4];  // BF16 pairs: columns 4g..4g+3 of tile 2*blk, then of tile 2*blk+1
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const v4f v = acc[i][2 * blk + t];
                        v2bf p0 = {(__bf16)v[0], (__bf16)v[1]}, p1 = {(__bf16)v[2], (__bf16)v[3]};
                        h[2 * t] = __builtin_bit_cast(uint32_t, p0);
                        h[2 * t + 1] = __builtin_bit_cast(uint32_t, p1);
                        *reinterpret_cast<uint2 *>(stage + r16 * PITCH + ((2 * blk + t) * 16 + 4 * g) * 2) = make_uint2(h[2 * t], h[2 * t + 1]);
                    }
                    // block amax on the magnitude bits: 8 values here, then the 3 other lanes of the row
                    uint32_t am = pk_max_u16(pk_max_u16(h[0] & 0x7FFF7FFFu, h[1] & 0x7FFF7FFFu),
                                             pk_max_u16(h[2] & 0x7FFF7FFFu, h[3] & 0x7FFF7FFFu));
                    am = umax(am & 0xFFFFu, am >> 16);
                    am = umax(am, (uint32_t)__shfl_xor((int)am, 16, 64));
                    am = umax(am, (uint32_t)__shfl_xor((int)am, 32, 64));
                    const uint32_t sb = scale_byte_from_bf16_bits(am);
                    const float sc = scale_operand(sb);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        uint32_t qt = cvt2_bf16(cvt2_bf16(0, h[2 * t], sc, false), h[2 * t + 1], sc, true);
                        if (sb >= 254) {  // NaN or Inf in the block: rare
                            if (sb == 0xFF) {
                                qt = 0x7F7F7F7Fu;
                            } else {
                                uint32_t f = 0;
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const uint32_t bits = (e & 1) ? h[2 * t + e / 2] >> 16 : h[2 * t + e / 2] & 0xFFFFu;
                                    f |= inf_byte_bf16(bits, (qt >> (8 * e)) & 0xFFu) << (8 * e);
                                }
                                qt = f;
                            }
                        }
                        q[2 * blk + t] = qt;
                    }
                    scales |= sb << (8 * blk);
                }
                __builtin_amdgcn_wave_barrier();  // the reads below see the other lanes' writes (LDS serves a wavefront in order)
#pragma unroll
                for (int t = 0; t < 16 * ROWB / 1024; ++t) {
                    const int lin = t * 1024 + lane * 16, row = lin / ROWB, colb = lin % ROWB;
                    const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * PITCH + colb);
                    *reinterpret_cast<uint4 *>(crow + (int64_t)(wm * Cfg::WM + row) * ldc_bytes + wn * ROWB + colb) = v;
                }
                __builtin_amdgcn_wave_barrier();  // the byte rows overwrite the area after these reads
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    *reinterpret_cast<uint32_t *>(stage + r16 * QPITCH + j * 16 + 4 * g) = q[j];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int t = 0; t < 16 * Cfg::WN / 1024; ++t) {
                    const int lin = t * 1024 + lane * 16, row = lin / Cfg::WN, colb = lin % Cfg::WN;
                    const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * QPITCH + colb);
                    *reinterpret_cast<uint4 *>(cq + (cur_tile.m0 + wm * Cfg::WM + i * 16 + row) * (int64_t)N + n_wave + colb) = v;
                }
                __builtin_amdgcn_wave_barrier();  // (the next row group overwrites the area after these reads)
                if (g == 0) {  // the TN/2 scale bytes of this row and wavefront: one dword or halfword
                    const int64_t nb = N / kBlock, b0 = n_wave / kBlock;
                    uint8_t *sp = TILED ? cs + (((m >> 6) * ((nb + 3) / 4) + (b0 >> 2)) * 64 + (m & 63)) * 4 + (b0 & 3)
                                        : cs + m * nb + b0;
                    if constexpr (TN / 2 == 4)
                        *reinterpret_cast<uint32_t *>(sp) = scales;
                    else
                        *reinterpret_cast<uint16_t *>(sp) = (uint16_t)scales;
                }
            } else {
                // Row group i of this wavefront (16 rows x WN columns) goes through a wavefront-private LDS area
                // so that it leaves as whole rows: a lane holds 4 consecutive columns of one row per MFMA tile,
                // and storing those directly costs one partial cache line per row and instruction (the address
                // unit of the compute unit then needs ~7 us per 256 x 256 tile, during which the matrix pipes
                // wait behind their own stores). Staged, every store instruction writes 1 KB of contiguous rows.
                constexpr int ROWB = Cfg::WN * ESZ;                            // bytes of one row of the wavefront's part
                constexpr int PITCH = ROWB + 32;                               // staged row pitch: spreads the rows over the banks
                constexpr int RPP = ROWB * 16 <= 4096 ? 16 : ROWB * 8 <= 4096 ? 8 : 4;  // rows per pass (at most 4 KB staged)
                static_assert(RPP * PITCH <= kStageBytes && (RPP * ROWB) % 1024 == 0, "staging area");
                uint8_t *stage = lds + Cfg::LDS_BYTES + wave * kStageBytes;
#pragma unroll
                for (int pass = 0; pass < 16 / RPP; ++pass) {
                    if (RPP == 16 || r16 / RPP == pass) {
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            const v4f v = acc[i][j];
                            uint8_t *dst = stage + (r16 % RPP) * PITCH + (j * 16 + 4 * g) * ESZ;
                            if constexpr (OUT_BF16) {
                                v2bf p0 = {(__bf16)v[0], (__bf16)v[1]}, p1 = {(__bf16)v[2], (__bf16)v[3]};
                                *reinterpret_cast<uint2 *>(dst) =
                                    make_uint2(__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1));
                            } else {
                                *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                            }
                        }
                    }
                    __builtin_amdgcn_wave_barrier();  // the reads below see the other lanes' writes (LDS serves a wavefront in order)
#pragma unroll
                    for (int t = 0; t < RPP * ROWB / 1024; ++t) {
                        const int lin = t * 1024 + lane * 16, row = lin / ROWB, colb = lin % ROWB;
                        const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * PITCH + colb);
                        const int m = wm * Cfg::WM + i * 16 + pass * RPP + row;  // inside the tile
                        if (GROUPED ? m < cur_tile.rows : !RAGGED || (m >= cur_tile.row_lo && wn * ROWB + colb >= cur_tile.col_lo * ESZ))
                            *reinterpret_cast<uint4 *>(crow + (int64_t)(wm * Cfg::WM + pass * RPP + row) * ldc_bytes +
                                                       wn * ROWB + colb) = v;
                    }
                    __builtin_amdgcn_wave_barrier();  // (the next pass overwrites the area after these reads)
                }
            }
            MXFP8_PIN();
        }
        if constexpr (FUSE_Q && !Q_ROW_ONLY) {
            uint8_t *stage = lds + Cfg::LDS_BYTES;
            const QuantLds qlds{stage, stage + kTile * kTile, stage + kTile * kTile + kTile * 4, nullptr, nullptr};
            for (int part = 0; part < (Cfg::BM / kTile) * (Cfg::BN / kTile); ++part) {
                __syncthreads();  // the tile of C is stored; the staging areas are free
                quantize_tile<true, (FUSE_Q & 1) != 0, (FUSE_Q & 2) != 0, TILED, 0>(
                    c, M, N, ldc_bytes, cq, cs, cqT, csT, nullptr, (uint32_t)(cur_tile.m0 / kTile + part / (Cfg::BN / kTile)),
                    (uint32_t)(cur_tile.n0 / kTile + part % (Cfg::BN / kTile)), tid, qlds);
            }
            __syncthreads();  // the next tile's rows are staged where the last piece was
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        cur_tile = next_tile;
    }
    MXFP8_WAIT_VMCNT(0);  // the redundant prefetches of the last steps must land before LDS is released
    if constexpr (GROUPED && Cfg::BM == 256 && Cfg::BN == 256) {
        using Quarter = StagedCfg<128, 128>;
        static_assert(Quarter::lds_bytes(TILED) <= Cfg::LDS_BYTES_PERSISTENT && Quarter::THREADS == Cfg::THREADS, "quarters on the same workgroup");
        if (tail.first(ntiles) < ntiles) {
            __syncthreads();  // the quarters' requests go where fragments and staged rows were read
            staged_grouped_rest<Quarter, OUT_BF16, TILED>(lds, a_q, a_s, b_q, b_s, M, N, K, c, ldc_bytes, tiles_n, tail, groups);
        }
    }
}

// Compute units of the current device.
static hipError_t compute_units(int &units)
{
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    units = cus > 0 ? cus : 1;
    return e;
}

// The same, and whether a launch may use all of them: a bound that is no smaller than the device is none.
static hipError_t compute_units(int max_workgroups, int &units, bool &all)
{
    const hipError_t e = compute_units(units);
    all = max_workgroups == 0 || max_workgroups >= units;
    return e;
}

// Number of workgroups of a persistent launch: one per compute unit of the current device, at most
// `max_workgroups` when the caller gives a positive bound, never more than there are tiles.
static hipError_t persistent_grid(int ntiles, int max_workgroups, int &grid)
{
    const hipError_t e = compute_units(grid);
    if (e != hipSuccess)
        return e;
    if (max_workgroups > 0 && max_workgroups < grid)
        grid = max_workgroups;
    if (ntiles < grid)
        grid = ntiles;
    return hipSuccess;
}

// The K-step schedule that spreads the requests over the step is the faster one on an MI355X wherever
// its spacing fits the tile (measured on the 8B-class layer shapes: +3 % over issuing them in bursts).
template <class Cfg> constexpr bool spread_fits()
{
    return 2 * Cfg::NB + 2 + 4 * (Cfg::NA - 1) < (Cfg::TN - 1) * Cfg::TM;
}
// The schedule of a configuration: the default spacing where it fits, else (two more requests per operand
// with MXFP4's second scale dword) A requests behind every 3rd MFMA pair, else bursts (0).
template <class Cfg> constexpr int sched_for()
{
    if (spread_fits<Cfg>())
        return MXFP8_GEMM_SCHED;
    if (2 * Cfg::NB + 2 + 3 * (Cfg::NA - 1) < (Cfg::TN - 1) * Cfg::TM)
        return 232;
    return 2 * Cfg::NB + 2 + 2 * (Cfg::NA - 1) < (Cfg::TN - 1) * Cfg::TM ? 222 : 0;
}

// Whether a problem runs on the persistent kernel with bm x bn tiles (K in bytes of an operand row): problems made of full
// tiles, and those of at least one 256-row tile whose rows of C end on 16 bytes. Everything else takes one workgroup per
// tile. (Ragged, BF16 out, tiled scales: [16000 x 6144 x 512] 108 us with one workgroup per tile, 67 us resident.)
static bool goes_resident(int bm, int bn, int M, int N, int K, const void *c, int64_t ldc_bytes, int esize)
{
    const bool full = M % bm == 0 && N % bn == 0;
    const bool ragged = bm == 256 && M >= bm && N >= bn && (int64_t)N * esize % 16 == 0;
    return (full || ragged) && K >= 2 * BK && reinterpret_cast<uintptr_t>(c) % 16 == 0 && ldc_bytes % 16 == 0 &&
           ldc_bytes * bm < (int64_t(1) << 31);
}

template <class Cfg, bool OUT_BF16, bool TILED>
static hipError_t launch_cfg(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                             int M, int N, int K, void *c, int64_t ldc, int max_workgroups, GemmTail tail, hipStream_t stream)
{
    const int tiles_m = (M + Cfg::BM - 1) / Cfg::BM, tiles_n = (N + Cfg::BN - 1) / Cfg::BN;
    const int64_t ldc_bytes = ldc * (OUT_BF16 ? 2 : 4);
    // 128-bit (FP32) / 64-bit (BF16) stores need every row start aligned; otherwise element stores
    const bool vec_store = (reinterpret_cast<uintptr_t>(c) % 16 == 0) && (ldc_bytes % 16 == 0);
    if (goes_resident(Cfg::BM, Cfg::BN, M, N, K, c, ldc_bytes, OUT_BF16 ? 2 : 4)) {
        const bool full = M % Cfg::BM == 0 && N % Cfg::BN == 0;
        int grid = 0;
        hipError_t e = persistent_grid(tiles_m * tiles_n, max_workgroups, grid);
        if (e != hipSuccess)
            return e;
        constexpr int sched = sched_for<Cfg>();
        auto kern = gemm_persistent_kernel<Cfg, OUT_BF16, TILED, sched != 0, 0, sched != 0 ? sched : MXFP8_GEMM_SCHED>;
        if constexpr (Cfg::BM == 256)
            if (!full)
                kern = gemm_persistent_kernel<Cfg, OUT_BF16, TILED, sched != 0, 0, sched != 0 ? sched : MXFP8_GEMM_SCHED, false, true>;
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                Cfg::LDS_BYTES_PERSISTENT);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Cfg::THREADS), Cfg::LDS_BYTES_PERSISTENT, stream, a_q, a_s, b_q, b_s, M, N, K,
                           static_cast<uint8_t *>(c), ldc_bytes, tiles_m, tiles_n, static_cast<uint8_t *>(nullptr),
                           static_cast<uint8_t *>(nullptr), static_cast<uint8_t *>(nullptr),
                           static_cast<uint8_t *>(nullptr), GemmGroups{nullptr, 0, 0, 0}, tail);
        return hipGetLastError();
    }
    auto kern = gemm_kernel<Cfg, OUT_BF16, TILED>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::LDS_BYTES);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(Cfg::THREADS), Cfg::LDS_BYTES, stream,
                       a_q, a_s, b_q, b_s, M, N, K, static_cast<uint8_t *>(c), ldc_bytes, tiles_m, tiles_n, vec_store,
                       GemmGroups{nullptr, 0, 0, 0});
    return hipGetLastError();
}

template <class Cfg>
static hipError_t launch_any(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s, int M,
                             int N, int K, void *c, bool c_bf16, bool tiled, int64_t ldc, int max_workgroups,
                             hipStream_t stream, GemmTail tail = {0, 0})
{
    if constexpr (Cfg::SCALED)
        if (tiled)
            return c_bf16 ? launch_cfg<Cfg, true, true>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, tail, stream)
                          : launch_cfg<Cfg, false, true>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, tail, stream);
    return c_bf16 ? launch_cfg<Cfg, true, false>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, tail, stream)
                  : launch_cfg<Cfg, false, false>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, tail, stream);
}

// ---- staged kernel (gemm_staged.h): everything that 256x256 tiles cannot spread over the chip -------------------
// What comes before a launch and can fail: a call of two launches has it done for both before the first one.
template <class Cfg, bool OUT_BF16, bool TILED, int TAIL> static hipError_t prepare_staged()
{
    constexpr int lds = Cfg::lds_bytes(TILED);
    if (lds <= 64 * 1024)  // what a launch may ask for by itself
        return hipSuccess;
    auto kern = gemm_staged_kernel<Cfg, OUT_BF16, TILED, TAIL>;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

// TAIL: of the 256x256 tiles that the resident kernel left, `tail_tiles` quarters at most (prepared by the caller)
template <class Cfg, bool OUT_BF16, bool TILED, int TAIL = kNoTail>
static hipError_t launch_staged_t(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s, int M, int N, int K,
                                  void *c, int64_t ldc, int max_workgroups, hipStream_t stream, GemmTail tail = {0, 0}, int tail_tiles = 0)
{
    constexpr int BM = TAIL == kNoTail ? Cfg::BM : 256, BN = TAIL == kNoTail ? Cfg::BN : 256;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int64_t ldc_bytes = ldc * (OUT_BF16 ? 2 : 4);
    const bool vec_store = (reinterpret_cast<uintptr_t>(c) % 16 == 0) && (ldc_bytes % 16 == 0);
    const int ntiles = TAIL == kNoTail ? tiles_m * tiles_n : tail_tiles;
    const int grid = max_workgroups > 0 && max_workgroups < ntiles ? max_workgroups : ntiles;
    if (TAIL == kNoTail) {
        const hipError_t e = prepare_staged<Cfg, OUT_BF16, TILED, TAIL>();
        if (e != hipSuccess)
            return e;
    }
    auto kern = gemm_staged_kernel<Cfg, OUT_BF16, TILED, TAIL>;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Cfg::THREADS), Cfg::lds_bytes(TILED), stream, a_q, a_s, b_q, b_s, M, N, K,
                       static_cast<uint8_t *>(c), ldc_bytes, tiles_m, tiles_n, vec_store, tail);
    return hipGetLastError();
}

template <class Cfg, int TAIL> static hipError_t prepare_staged_cfg(bool c_bf16, bool tiled)
{
    if constexpr (Cfg::SCALED)
        if (tiled)
            return c_bf16 ? prepare_staged<Cfg, true, true, TAIL>() : prepare_staged<Cfg, false, true, TAIL>();
    return c_bf16 ? prepare_staged<Cfg, true, false, TAIL>() : prepare_staged<Cfg, false, false, TAIL>();
}

template <class Cfg, int TAIL = kNoTail>
static hipError_t launch_staged_cfg(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s, int M, int N, int K,
                                    void *c, bool c_bf16, bool tiled, int64_t ldc, int max_workgroups, hipStream_t stream,
                                    GemmTail tail = {0, 0}, int tail_tiles = 0)
{
    if constexpr (Cfg::SCALED)
        if (tiled)
            return c_bf16 ? launch_staged_t<Cfg, true, true, TAIL>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, stream, tail, tail_tiles)
                          : launch_staged_t<Cfg, false, true, TAIL>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, stream, tail, tail_tiles);
    return c_bf16 ? launch_staged_t<Cfg, true, false, TAIL>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, stream, tail, tail_tiles)
                  : launch_staged_t<Cfg, false, false, TAIL>(a_q, a_s, b_q, b_s, M, N, K, c, ldc, max_workgroups, stream, tail, tail_tiles);
}

// Which tile: an estimate of the time, what a launch costs around its K loop plus (rounds of tiles over the compute units)
// x (K steps) x (time of a step), from measurements on an MI355X (MXFP8, row-major scales, BF16 out, us; 256-row tiles on the
// resident kernel from 256 rows on, else one workgroup per tile):
//                          256x256 256x192 128x128 128x64 64x128  64x64  32x64  32x32
//   [2048 x 6144 x 4096]      50.2    48.8    54.8   74.3   75.9   81.5  124.0  171.2
//   [2048 x 3072 x 4096]      46.0    40.5    35.3   38.6   39.5   43.5   67.9   90.1
//   [1000 x 2880 x 5760]      61.1    57.3    25.2   35.3   36.1   32.7   48.7   64.5
//   [512 x 4096 x 4096]       44.4    39.2    17.9   14.7   15.1   17.3   25.1   32.5
//   [128 x 4096 x 4096]       43.6    36.9    14.9   11.4   13.9    9.0    8.9   10.0
//   [48 x 6144 x 4096]        41.8    32.8    15.0   11.7   11.8    9.1    9.5    9.6
//   [384 x 896 x 512]         12.2    10.4     6.2    4.9    4.9    4.2    3.8    3.9
//   [304 x 704 x 640]         13.2    11.1     6.3    5.0    5.0    4.2    3.8    3.6
//   [16 x 1024 x 2048]        23.1    18.6     9.4    7.5    7.6    5.9    5.6    4.9
// Other operands keep the order of the tiles, or nearly: the same operand bytes take 0.9 of the time with tiled scales, 0.85 as
// BF16, 1.2 as MXFP4 with tiled scales ([1000 x 2880], 45 steps, 128x128: 22.3, 21.3, 31.5; 64x64: 28.3, 26.7, 32.1).
// A 128x128 step takes longer where all units of the device have several tiles (all of them fetch all the time); under a
// bound, also one of 200 or 250 of 256 units, the shorter time was the better estimate. The 256x256 tiles of the kernels
// above take 1.5 us per step, but share each fetched byte among twice as many matrix instructions. Where they cannot go
// resident, their prologue and epilogue are paid in every round and a step is slower ([137 x 74069 x 4864], BF16 out, tiled:
// 153.8 us as one-tile 256x256 workgroups, 138.4 as staged 64x128 tiles; [6144 x 6922 x 3456]: 211.6 us, 235.0 as staged
// 128x128 tiles).
// Tiles of 96 columns fill a round that 128 leave a quarter empty, in one run with operands that rotate (tiled scales, BF16 out):
//                          128x128 128x96 128x64 64x96 64x64
//   [1000 x 2880 x 5760]      30.1   27.9   35.8  37.0  32.6   (34.4, 32.6, 41.5, 43.3, 38.2 with row-major scales)
//   [1000 x 2880 x 2048]      11.2   11.7   14.2  14.2  12.3
//   [200 x 5120 x 8192]       36.6   31.7   27.7  23.5  25.5
//   [200 x 5120 x 2048]       10.2   10.7    8.0   8.0   8.6
//   [850 x 1200 x 4096]       16.5   15.1   12.3  11.4  14.2   (FP32 out)
// Their own numbers are those that lose least against the other tiles over 780 products of 33 .. 2400 rows and 6 .. 72 steps, with
// operands that rotate and that stay: chosen for 184 of them, 6 % faster there, one slower by more than 2 % both ways (5 %). Several
// rounds of 64x96 tiles cost more than the smaller step shows ([768 x 6144 x 2048] as 768 of them 26.4 us, 20.8 as 64x64 tiles).
// A ring of eight K steps for the small tiles was no faster (64x64: 8.7 -> 9.0 us at [128 x 4096 x 4096], 18.1 -> 19.3 at [512 x
// 4096 x 4096]): workgroups side by side on a unit hide more than a deeper ring does, and LDS is what they need.
// units: compute units that the launch may use; all_units: it may use all of them; route(bm, bn): how 256-row tiles would run.
enum class Tile { k256, k256_tail, k256x192, k128, k128x96, k128x64, k64x128, k64x96, k64, k32x64, k32 };
enum class Route { resident, one_tile, none };
struct TileOption {
    Tile tile;
    int bm, bn;
    double around_us, round_us, step_us, step_us_full;
    int64_t tiles(int64_t M, int64_t N) const { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
    int64_t rounds(int64_t M, int64_t N, int64_t units) const { return (tiles(M, N) + units - 1) / units; }
};
template <class F> static TileOption choose_tile(int64_t M, int64_t N, int64_t KT, int64_t units, bool all_units, F route)
{
    static const TileOption options[] = {{Tile::k256, 256, 256, 5.0, 0, 1.45, 1.45}, {Tile::k256x192, 256, 192, 5.0, 0, 1.2, 1.2},
                                         {Tile::k128, 128, 128, 4.0, 0, 0.43, 0.55}, {Tile::k128x96, 128, 96, 5.2, 0, 0.395, 0.50}, {Tile::k128x64, 128, 64, 3.5, 0, 0.32, 0.36},
                                         {Tile::k64x128, 64, 128, 3.5, 0, 0.32, 0.36}, {Tile::k64x96, 64, 96, 3.5, 1.3, 0.265, 0.32}, {Tile::k64, 64, 64, 2.6, 0, 0.215, 0.215},
                                         {Tile::k32x64, 32, 64, 2.4, 0, 0.19, 0.19}, {Tile::k32, 32, 32, 2.2, 0, 0.165, 0.165}};
    static const TileOption one_tile[] = {{Tile::k256, 256, 256, 3.0, 1.5, 1.5, 1.5}, {Tile::k256x192, 256, 192, 2.0, 2.5, 1.22, 1.22}};
    TileOption best = options[0];
    double least = 1e30;
    for (TileOption o : options) {
        if (o.bm == 256) {
            const Route r = route(o.bm, o.bn);
            if (r == Route::none)
                continue;
            if (r == Route::one_tile)
                o = one_tile[o.tile == Tile::k256 ? 0 : 1];
        }
        const double step = o.tiles(M, N) > units && all_units ? o.step_us_full : o.step_us;
        const double us = o.around_us + (double)o.rounds(M, N, units) * (o.round_us + (double)KT * step);
        if (us < least) {
            least = us;
            best = o;
        }
    }
    // 256x256 tiles for the full rounds, a rest of few tiles as quarters on the staged kernel, in a launch of its own (8 us around
    // its K loop), where that is expected to save 4 % (with less, [12544 x 2688 x 6528] took 180 us for 172 as 256x192 tiles). A round
    // of few 256x256 tiles takes 0.7 us per step, a round of 128x128 tiles 0.43. In us, whole | with the rest as
    // quarters: [4352 x 4096 x 4096] (272 tiles, BF16 out, tiled) 73.4 | 70.2, [5376 x 3328 x 8192] 133.5 | 123.5, FP32 out, row-major
    // 156.9 | 138.2; but [4352 x 4096 x 1024] 27.2 | 29.0, [7828 x 4400 x 4480] (46 more than two rounds) 129.1 | 134.3.
    const TileOption &whole = options[0], &quarter = options[2];  // 256x256, 128x128
    const int64_t n = whole.tiles(M, N), rest = n % units;
    if (all_units && n > units && rest > 0 && 8 * rest <= units && KT >= 28 && route(256, 256) == Route::resident &&
        1.04 * (whole.around_us + (double)(n / units * KT) * whole.step_us + 8.0 + (double)KT * quarter.step_us) < least) {
        best = whole;
        best.tile = Tile::k256_tail;
    }
    return best;
}

// K in bytes of an operand row. The bound on workgroups applies to problems made of full 256x256 tiles (128x128 ones where there
// are fewer than 128 of the large) whose rows of C are aligned, and the tile is chosen for the units it leaves; everything
// else ignores it. [2048 x 2048 x 4096] on 64 workgroups (row-major scales): resident 128x128 tiles 102.5 us, staged 128x128
// tiles 60.5 us, resident 256x256 tiles 45.7 us; [512 x 6144 x 4096] on 32: 150.5, 87, 256x192 tiles 72 us. The staged kernel fills a ring of four K steps before it starts.
template <int FMT, bool A5, bool B5>
static hipError_t launch_product(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s, int M, int N, int K,
                                 void *c, bool c_bf16, bool tiled, int64_t ldc, int max_workgroups, hipStream_t stream)
{
    const bool many = (int64_t)((M + 255) / 256) * ((N + 255) / 256) >= 128;
    const int full = many ? 256 : 128;
    const int esize = c_bf16 ? 2 : 4;
    const int64_t ldc_bytes = ldc * esize;
    const bool whole = M % full == 0 && N % full == 0 && goes_resident(full, full, M, N, K, c, ldc_bytes, esize);
    if (!whole)
        max_workgroups = 0;
    // 256-row tiles keep a bound only on the resident kernel (rows of C 8 MiB and more apart do not fit its offsets)
    auto route = [&](int bm, int bn) {
        return goes_resident(bm, bn, M, N, K, c, ldc_bytes, esize) ? Route::resident : max_workgroups == 0 ? Route::one_tile : Route::none;
    };
    const int KT = K / BK;
    Tile tile = Tile::k256;
    int units = 0;
    bool two_buffers = K < 4 * BK && !many;  // 128x128 tiles on the resident or the one-tile kernel instead of the staged one
    if (K >= 4 * BK) {
        bool all_units = false;
        const hipError_t e = compute_units(max_workgroups, units, all_units);
        if (e != hipSuccess)
            return e;
        units = all_units ? units : max_workgroups;
        const TileOption o = choose_tile(M, N, KT, units, all_units, route);
        tile = o.tile;
        const int64_t tiles128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
        const bool staged = tile != Tile::k256 && tile != Tile::k256x192 && tile != Tile::k256_tail;
        if (staged && goes_resident(128, 128, M, N, K, c, ldc_bytes, esize)) {
            // Few K steps and several tiles per workgroup: the resident kernel fetches the next tile under the epilogue of
            // the last, the staged one starts anew. [896 x 2688 x 512] on 40 workgroups (row-major scales): staged 18.0 us,
            // resident 15.7; from 11 steps on the staged kernel wins ([2304 x 2176 x 1408] on 40: 49.8 against 57.8), with
            // row-major MXFP4 scales always ([1024 x 4352 x 1280]: 11.0, 13.4), and where half the units would get no tile
            // ([384 x 1408 x 1024] MXFP4 on 100: 5.8, 6.6).
            two_buffers = KT <= (tile == Tile::k128 ? 10 : 6) && o.rounds(M, N, units) >= 2 && (FMT != kFmtFp4 || tiled) &&
                          2 * tiles128 >= units;
        } else if (staged && max_workgroups == 0 && tile != Tile::k32x64 && tile != Tile::k32) {
            // Two of the one-tile kernel's 128x128 workgroups fit a unit, so what takes the staged kernel two rounds runs side
            // by side. Not with row-major scales (a cache line per row and request), FP32 output (its direct stores) or few
            // rows, and not before the second place of a quarter of the units is filled. BF16 out, tiled: [2064 x 3528 x 5376]
            // MXFP4 33.5 us staged, 28.8 here; [2254 x 2584 x 1280] MXFP8 17.1, 15.4; but [651 x 5566 x 16640] MXFP4 (264
            // tiles) 67.3 and 71.3, and [564 x 6688 x 1024] MXFP4, FP32 out, 9.1 and 12.8.
            two_buffers = (FMT == kFmtBf16 || tiled) && c_bf16 && M > 64 && N > 64 && 4 * tiles128 > 5 * units && tiles128 <= 2 * units &&
                           (tile == Tile::k128 || KT >= 8);
        }
    }
    if (two_buffers)
        return launch_any<GemmCfg<128, 128, 2, 2, FMT, A5, B5>>(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled, ldc, max_workgroups, stream);
#define MXFP8_STAGED(BM, BN) \
    return launch_staged_cfg<StagedCfg<BM, BN, FMT, A5, B5>>(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled, ldc, max_workgroups, stream)
    switch (tile) {
    case Tile::k128: MXFP8_STAGED(128, 128);
    case Tile::k128x96: MXFP8_STAGED(128, 96);
    case Tile::k64x96: MXFP8_STAGED(64, 96);
    case Tile::k128x64: MXFP8_STAGED(128, 64);
    case Tile::k64x128: MXFP8_STAGED(64, 128);
    case Tile::k64: MXFP8_STAGED(64, 64);
    case Tile::k32x64: MXFP8_STAGED(32, 64);
    case Tile::k32: MXFP8_STAGED(32, 32);
    case Tile::k256x192:
        return launch_any<GemmCfg<256, 192, 2, 2, FMT, A5, B5>>(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled, ldc, max_workgroups, stream);
    case Tile::k256_tail: {
        using Quarter = StagedCfg<128, 128, FMT, A5, B5>;
        const GemmTail tail = {units, units};
        const int n = ((M + 255) / 256) * ((N + 255) / 256);
        hipError_t e = prepare_staged_cfg<Quarter, kTailPlain>(c_bf16, tiled);
        if (e == hipSuccess)
            e = launch_any<GemmCfg<256, 256, 2, 2, FMT, A5, B5>>(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled, ldc, 0, stream, tail);
        return e != hipSuccess ? e : launch_staged_cfg<Quarter, kTailPlain>(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled, ldc, 0, stream, tail,
                                                                            4 * (n - tail.first(n)));
    }
    case Tile::k256: break;
    }
#undef MXFP8_STAGED
    return launch_any<GemmCfg<256, 256, 2, 2, FMT, A5, B5>>(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled, ldc, max_workgroups, stream);
}

hipError_t launch_gemm(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s, int64_t M,
                       int64_t N, int64_t K, void *c, bool c_bf16, bool tiled_scales, int64_t ldc, int max_workgroups,
                       hipStream_t stream)
{
    return launch_product<kFmtFp8, false, false>(a_q, a_s, b_q, b_s, (int)M, (int)N, (int)K, c, c_bf16, tiled_scales, ldc,
                                                 max_workgroups, stream);
}

// Grouped product over expert-sorted rows of A (see GemmGroups). Always the persistent kernel: N a multiple of
// the tile (256 when the problem is large and N allows it, else 128), K >= 2 steps, C vector-storable; returns
// hipErrorInvalidConfiguration (nothing launched) otherwise. The host does not know the number of tiles: the
// grid is one workgroup per compute unit (or max_workgroups), capped by the largest number there can be.
template <class Cfg, bool OUT_BF16, bool TILED>
static hipError_t launch_grouped_cfg(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                                     const GemmGroups &groups, int M, int N, int K, void *c, int64_t ldc,
                                     int max_workgroups, hipStream_t stream)
{
    const int64_t ldc_bytes = ldc * (OUT_BF16 ? 2 : 4);
    const bool vec_store = (reinterpret_cast<uintptr_t>(c) % 16 == 0) && (ldc_bytes % 16 == 0);
    if (N % Cfg::BN || K < 2 * BK || !vec_store || ldc_bytes * Cfg::BM >= (int64_t(1) << 31))
        return hipErrorInvalidConfiguration;
    const int tiles_n = N / Cfg::BN;
    const int64_t most_tiles = ((int64_t)(M + Cfg::BM - 1) / Cfg::BM + groups.count) * tiles_n;
    int units = 0, grid = 0;
    bool all_units = false;
    hipError_t e = compute_units(max_workgroups, units, all_units);
    if (e == hipSuccess)
        e = persistent_grid((int)(most_tiles < 0x7FFFFFFF ? most_tiles : 0x7FFFFFFF), max_workgroups, grid);
    if (e != hipSuccess)
        return e;
    // Where there are more tiles than units, few tiles of an unfilled last round are computed as quarters, like those of a plain
    // product (choose_tile), which has other tiles to choose from. Only the device knows how many there are, so the same workgroups
    // go on with them. In us, whole | as quarters in a launch of their own | this way: [8192 x 2048 x 5632] in 8 experts, 272 tiles,
    // 134.8 | 104.6 | 100.6; [8192 x 2048 x 2048], 288 tiles, 59.3 | 49.7 | 46.9; and where there is no such rest [4096 x 4096 x
    // 2048], 304 tiles, 57.4 | 59.3 | 57.6, [8192 x 2048 x 2048], 256 tiles, 38.0 | 39.3 | 37.6 (BF16 out, both scale layouts).
    GemmTail tail = {0, 0};
    if (Cfg::BM == 256 && all_units && most_tiles > grid && K >= 16 * BK)
        tail = {grid, K >= 28 * BK ? grid / 4 : grid / 8};
    auto kern = gemm_persistent_kernel<Cfg, OUT_BF16, TILED, spread_fits<Cfg>(), 0, MXFP8_GEMM_SCHED, true>;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            Cfg::LDS_BYTES_PERSISTENT);
    if (e != hipSuccess)
        return e;
    uint8_t *none = nullptr;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Cfg::THREADS), Cfg::LDS_BYTES_PERSISTENT, stream, a_q, a_s, b_q, b_s, M, N, K,
                       static_cast<uint8_t *>(c), ldc_bytes, 0, tiles_n, none, none, none, none, groups, tail);
    return hipGetLastError();
}

// Weight-gradient form of the grouped product: resident workgroups where 256x256 tiles go resident and there are no more experts
// than those sort (see gemm_persistent_kernel, KGROUPED), else one workgroup per (expert, tile) (gemm_kernel, KGROUPED).
template <class Cfg, bool OUT_BF16, bool TILED>
static hipError_t launch_kgrouped_cfg(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                                      const GemmGroups &groups, int M, int N, int K, void *c, int64_t ldc, hipStream_t stream)
{
    const int tiles_m = (M + Cfg::BM - 1) / Cfg::BM, tiles_n = (N + Cfg::BN - 1) / Cfg::BN;
    const int64_t ldc_bytes = ldc * (OUT_BF16 ? 2 : 4);
    const bool vec_store = (reinterpret_cast<uintptr_t>(c) % 16 == 0) && (ldc_bytes % 16 == 0) && ((int64_t)M * ldc_bytes) % 16 == 0;
    const int64_t grid = (int64_t)groups.count * tiles_m * tiles_n;
    if (grid > 0x7FFFFFFF)
        return hipErrorInvalidConfiguration;
    if constexpr (Cfg::BM == 256) {
        if (groups.count <= kMostKExperts && goes_resident(Cfg::BM, Cfg::BN, M, N, K, c, ldc_bytes, OUT_BF16 ? 2 : 4)) {
            const bool full = M % Cfg::BM == 0 && N % Cfg::BN == 0;
            int units = 0;
            hipError_t e = persistent_grid((int)grid, 0, units);
            if (e != hipSuccess)
                return e;
            constexpr int sched = sched_for<Cfg>(), lds = Cfg::LDS_BYTES_PERSISTENT + kMostKExperts * (int)sizeof(KExpert);
            static_assert(lds <= 160 * 1024, "LDS of a unit");
            auto kern = full ? gemm_persistent_kernel<Cfg, OUT_BF16, TILED, true, 0, sched, false, false, true>
                             : gemm_persistent_kernel<Cfg, OUT_BF16, TILED, true, 0, sched, false, true, true>;
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess)
                return e;
            uint8_t *none = nullptr;
            hipLaunchKernelGGL(kern, dim3((unsigned)units), dim3(Cfg::THREADS), lds, stream, a_q, a_s, b_q, b_s, M, N, K,
                               static_cast<uint8_t *>(c), ldc_bytes, tiles_m, tiles_n, none, none, none, none, groups, GemmTail{0, 0});
            return hipGetLastError();
        }
    }
    auto kern = gemm_kernel<Cfg, OUT_BF16, TILED, true>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::LDS_BYTES);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Cfg::THREADS), Cfg::LDS_BYTES, stream, a_q, a_s, b_q, b_s, M, N, K,
                       static_cast<uint8_t *>(c), ldc_bytes, tiles_m, tiles_n, vec_store, groups);
    return hipGetLastError();
}

hipError_t launch_gemm_kgrouped(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                                const int32_t *group_ends, int groups, int64_t M, int64_t N, int64_t K, void *c, bool c_bf16,
                                bool tiled_scales, int64_t ldc, hipStream_t stream)
{
    using Big = GemmCfg<256, 256, 2, 2>;
    using Small = GemmCfg<128, 128, 2, 2>;
    const GemmGroups g{group_ends, groups, 0, 0};
    const bool big = ((M + 255) / 256) * ((N + 255) / 256) * groups >= 128;
    const int m = (int)M, n = (int)N, k = (int)K;
#define MXFP8_KGROUPED(CFG)                                                                                        \
    (c_bf16 ? (tiled_scales ? launch_kgrouped_cfg<CFG, true, true>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, stream)   \
                            : launch_kgrouped_cfg<CFG, true, false>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, stream)) \
            : (tiled_scales ? launch_kgrouped_cfg<CFG, false, true>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, stream)  \
                            : launch_kgrouped_cfg<CFG, false, false>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, stream)))
    return big ? MXFP8_KGROUPED(Big) : MXFP8_KGROUPED(Small);
#undef MXFP8_KGROUPED
}

hipError_t launch_gemm_grouped(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                               const int32_t *group_ends, int groups, int64_t b_group_bytes, int64_t bs_group_bytes,
                               int64_t M, int64_t N, int64_t K, void *c, bool c_bf16, bool tiled_scales, int64_t ldc,
                               int max_workgroups, hipStream_t stream)
{
    using Big = GemmCfg<256, 256, 2, 2>;
    using Small = GemmCfg<128, 128, 2, 2>;
    const GemmGroups g{group_ends, groups, b_group_bytes, bs_group_bytes};
    const bool big = N % 256 == 0 && ((M + 255) / 256) * (N / 256) >= 128;
    const int m = (int)M, n = (int)N, k = (int)K;
#define MXFP8_GROUPED(CFG)                                                                                                     \
    (c_bf16 ? (tiled_scales ? launch_grouped_cfg<CFG, true, true>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, max_workgroups, stream)   \
                            : launch_grouped_cfg<CFG, true, false>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, max_workgroups, stream)) \
            : (tiled_scales ? launch_grouped_cfg<CFG, false, true>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, max_workgroups, stream)  \
                            : launch_grouped_cfg<CFG, false, false>(a_q, a_s, b_q, b_s, g, m, n, k, c, ldc, max_workgroups, stream)))
    return big ? MXFP8_GROUPED(Big) : MXFP8_GROUPED(Small);
#undef MXFP8_GROUPED
}

// MXFP8 product with the element format of each operand chosen by the caller (E4M3 or E5M2: Section 3.2.2).
hipError_t launch_gemm_elements(const uint8_t *a_q, const uint8_t *a_s, bool a_e5m2, const uint8_t *b_q, const uint8_t *b_s,
                                bool b_e5m2, int64_t M, int64_t N, int64_t K, void *c, bool c_bf16, bool tiled_scales, int64_t ldc,
                                int max_workgroups, hipStream_t stream)
{
    const int m = (int)M, n = (int)N, k = (int)K;
    if (a_e5m2)
        return b_e5m2 ? launch_product<kFmtFp8, true, true>(a_q, a_s, b_q, b_s, m, n, k, c, c_bf16, tiled_scales, ldc, max_workgroups, stream)
                      : launch_product<kFmtFp8, true, false>(a_q, a_s, b_q, b_s, m, n, k, c, c_bf16, tiled_scales, ldc, max_workgroups, stream);
    if (b_e5m2)
        return launch_product<kFmtFp8, false, true>(a_q, a_s, b_q, b_s, m, n, k, c, c_bf16, tiled_scales, ldc, max_workgroups, stream);
    return launch_gemm(a_q, a_s, b_q, b_s, M, N, K, c, c_bf16, tiled_scales, ldc, max_workgroups, stream);
}

// Product of two MXFP4 operands (Table 1: E2M1 elements, two per byte), [M x K/2] and [N x K/2] bytes with K/32
// scale bytes per row: the same block-scaled sum (Section 2, Appendix A.3) on the 4-bit form of the scaled matrix
// instruction. K is counted in elements here and in bytes inside the kernels.
hipError_t launch_gemm_fp4(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s, int64_t M,
                           int64_t N, int64_t K, void *c, bool c_bf16, bool tiled_scales, int64_t ldc, int max_workgroups,
                           hipStream_t stream)
{
    return launch_product<kFmtFp4, false, false>(a_q, a_s, b_q, b_s, (int)M, (int)N, (int)(K / 2), c, c_bf16, tiled_scales, ldc,
                                                 max_workgroups, stream);
}

// Product of two BF16 operands, [M x K] and [N x K], both K-contiguous, FP32 accumulation: the GEMM of the
// simulated path (Section 3.1). Same kernels as the MXFP8 product with the BF16 matrix instruction and no
// scales; K is counted in elements here and in bytes inside the kernels.
hipError_t launch_gemm_bf16(const uint8_t *a, const uint8_t *b, int64_t M, int64_t N, int64_t K, void *c, bool c_bf16,
                            int64_t ldc, int max_workgroups, hipStream_t stream)
{
    const uint8_t *none = nullptr;
    return launch_product<kFmtBf16, false, false>(a, none, b, none, (int)M, (int)N, (int)(2 * K), c, c_bf16, false, ldc, max_workgroups, stream);
}

// GEMM with BF16 output and MXFP8 copies of that output (axis bit 0: row-wise, bit 1: column-wise) from
// the same call. Full tiles only: returns hipErrorInvalidConfiguration (nothing launched) when M or N is not a multiple of
// the tile (256 when the problem has at least 128 such tiles, else 128) or K has fewer than two steps.
template <class Cfg, bool TILED, int AXIS>
static hipError_t launch_fused_cfg(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                                   int M, int N, int K, void *c, int64_t ldc, uint8_t *cq, uint8_t *cs, uint8_t *cqT,
                                   uint8_t *csT, int max_workgroups, hipStream_t stream)
{
    const int64_t ldc_bytes = ldc * 2;
    const int tiles_m = M / Cfg::BM, tiles_n = N / Cfg::BN;
    auto kern = gemm_persistent_kernel<Cfg, true, TILED, spread_fits<Cfg>(), AXIS>;
    int grid = 0;
    hipError_t e = persistent_grid(tiles_m * tiles_n, max_workgroups, grid);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                Cfg::LDS_BYTES_PERSISTENT);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Cfg::THREADS), Cfg::LDS_BYTES_PERSISTENT, stream, a_q, a_s, b_q, b_s, M, N, K,
                       static_cast<uint8_t *>(c), ldc_bytes, tiles_m, tiles_n, cq, cs, cqT, csT, GemmGroups{nullptr, 0, 0, 0}, GemmTail{0, 0});
    return hipGetLastError();
}

template <class Cfg, bool TILED, class... Args> static hipError_t launch_fused_axis(int axis, Args... args)
{
    switch (axis) {
    case 1: return launch_fused_cfg<Cfg, TILED, 1>(args...);
    case 2: return launch_fused_cfg<Cfg, TILED, 2>(args...);
    default: return launch_fused_cfg<Cfg, TILED, 3>(args...);
    }
}

// Which way (both measured on an MI355X in one run, graph replays over three sets of operands, tiled scales, us: one kernel |
// product, then quantizer, by K steps):
//   row copy     tiles256          2             8             32
//   [2816 x 3072]     132    19.9 |  19.4   26.0 |  23.1   50.9 |  43.5
//   [3328 x 4096]     208    20.0 |  21.2   26.9 |  28.0   53.7 |  55.5
//   [4352 x 4096]     272    33.4 |  29.9   46.0 |  38.1  100.2 |  77.3
//   [6144 x 4096]     384    33.7 |  33.0   47.4 |  46.4  105.4 | 103.2
//   [8192 x 4096]     512    35.4 |  38.2   52.0 |  55.2  120.2 | 119.0
//   [8192 x 14336]   1792   105.8 | 108.9  165.8 | 171.1  395.2 | 398.2   (row-major scales 105.6 | 116.4, 167.7 | 181.4, 429.2 | 433.7)
//   both copies
//   [2816 x 3072]     132    28.2 |  21.5   34.2 |  25.2   59.2 |  45.7
//   [8192 x 4096]     512    60.0 |  44.3   77.7 |  60.3  141.3 | 123.4
//   [8192 x 14336]   1792   190.5 | 134.5  246.9 | 201.1  454.1 | 430.9
//   row copy     tiles128          2             4             8            12            16
//   [512 x 1024]       32     7.3 |   9.1    8.2 |   7.7    9.9 |   8.2   11.9 |   9.2   14.2 |  10.2
//   [1024 x 1536]      96     7.6 |  10.4    8.7 |  10.3   11.3 |  11.4   13.6 |  12.2   16.0 |  12.9
//   [1280 x 2048]     160     8.1 |  11.3    9.2 |  12.8   12.0 |  13.3   14.0 |  14.5   16.4 |  15.7
//   [2048 x 2048]     256     8.8 |  13.4   10.1 |  12.7   12.7 |  15.5   15.4 |  16.2   18.0 |  17.9   (both 11.3 | 14.3 .. 20.1 | 19.7)
//   [1920 x 2432]     285    13.4 |  15.2   15.6 |  16.6   19.5 |  18.3   23.7 |  21.3   28.0 |  24.2   (both 17.2 | 16.7 .. 31.7 | 25.9)
//   [2560 x 2560]     400    13.6 |  15.5   15.6 |  17.3   19.4 |  20.9   24.0 |  26.2   29.1 |  27.0   (both 17.8 | 17.6 .. 33.1 | 29.0)
// An epilogue that converts keeps the matrix pipes of its unit idle, and it ties the product to 256x256 (128x128) tiles; the
// quantizer reads C from the caches at the rate of the memory. So of large problems the column copy is left to the quantizer, and
// the row copy, which the epilogue makes straight from the accumulators, where the tiles fill three quarters of their rounds or
// less. Small problems stay in one kernel while the second launch costs more than the smaller tiles of the plain product save:
// the more tiles, the more K steps, up to a full round; in a second round all of it when both copies are wanted. Under a bound on
// workgroups neither way wins ([4096 x 14336 x 4096], both copies, on 64: 723.9 | 719.2; [2816 x 3072 x 512], row copy, on
// 32: 80.1 | 92.7; [2048 x 2048 x 1024], both, on 192: 19.8 | 23.8): one kernel.
static bool fused_in_one_kernel(bool big, int axis, int64_t tiles, int64_t steps, int64_t units)
{
    const int64_t rounds = (tiles + units - 1) / units;
    if (big)
        return axis == 1 && 4 * tiles > 3 * rounds * units;
    if (rounds == 1)
        return steps <= std::min<int64_t>(12, std::max<int64_t>(3, 20 * tiles / units));
    return axis != 3 && steps <= (2 * tiles < 3 * units ? 7 : 12);
}

hipError_t launch_gemm_fused(const uint8_t *a_q, const uint8_t *a_s, const uint8_t *b_q, const uint8_t *b_s,
                             int64_t M, int64_t N, int64_t K, void *c, int64_t ldc, int axis, uint8_t *cq,
                             uint8_t *cs, uint8_t *cqT, uint8_t *csT, bool tiled_scales, int max_workgroups,
                             hipStream_t stream)
{
    using Big = GemmCfg<256, 256, 2, 2>;
    using Small = GemmCfg<128, 128, 2, 2>;
    const int64_t tiles256 = ((M + 255) / 256) * ((N + 255) / 256);
    const bool big = tiles256 >= 128;
    const int m = (int)M, n = (int)N, k = (int)K, bm = big ? 256 : 128;
    if (M % bm || N % bm || K < 2 * BK || ldc * 2 * bm >= (int64_t(1) << 31))
        return hipErrorInvalidConfiguration;
    int units = 0;
    bool all_units = false;
    hipError_t e = compute_units(max_workgroups, units, all_units);
    if (e != hipSuccess)
        return e;
    if (all_units) {
        if (!fused_in_one_kernel(big, (int)axis, big ? tiles256 : (M / 128) * (N / 128), K / BK, units)) {
            e = launch_gemm(a_q, a_s, b_q, b_s, M, N, K, c, true, tiled_scales, ldc, 0, stream);
            return e != hipSuccess ? e : launch_quantize(c, true, M, N, ldc, axis, cq, cs, cqT, csT, tiled_scales, 0, stream);
        }
    }
    if (big)
        return tiled_scales ? launch_fused_axis<Big, true>(axis, a_q, a_s, b_q, b_s, m, n, k, c, ldc, cq, cs, cqT, csT, max_workgroups, stream)
                            : launch_fused_axis<Big, false>(axis, a_q, a_s, b_q, b_s, m, n, k, c, ldc, cq, cs, cqT, csT, max_workgroups, stream);
    return tiled_scales ? launch_fused_axis<Small, true>(axis, a_q, a_s, b_q, b_s, m, n, k, c, ldc, cq, cs, cqT, csT, max_workgroups, stream)
                        : launch_fused_axis<Small, false>(axis, a_q, a_s, b_q, b_s, m, n, k, c, ldc, cq, cs, cqT, csT, max_workgroups, stream);
}

}  // namespace mxfp8
