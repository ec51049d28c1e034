// What the product kernels share: operand formats, the order of the output tiles, one K step of one 16x16 output
// tile, wait counts. The register layout of the matrix instructions is described in gemm.hip.
#pragma once
#include "mxfp8_device.h"

namespace mxfp8 {

constexpr int BK = 128;  // K bytes per step = 4 scale blocks = one MFMA
constexpr int kStageBytes = 4608;  // per-wavefront LDS area of the persistent kernel's epilogue (16 rows x (256 + 32) bytes)

// Operand formats. kFmtFp8: MXFP8 operands with their scale bytes (the method itself), 128 elements and 4 scale
// blocks per 128-byte K step. kFmtBf16: plain BF16 operands, 64 per K step, no scales (the product of the
// simulated path of Section 3.1). kFmtFp4: MXFP4 operands (Table 1), two E2M1 codes per byte: 256 elements and
// 8 scale blocks (two scale dwords per row) per K step. Everything about tiles, buffers, data requests and the
// schedule is counted in BYTES of a K-contiguous operand row and is the same for all three.
constexpr int kFmtFp8 = 0, kFmtBf16 = 1, kFmtFp4 = 2;
// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2. Renumber them so
// that consecutive logical ids run on the same XCD, then walk the tile grid in column panels of
// `PANEL` tiles so that the workgroups resident on one XCD share A rows and B rows in its L2.
__device__ __forceinline__ int xcd_logical_id(int bid, int nblocks)
{
    constexpr int XCDS = 8;
    const int full = (nblocks / XCDS) * XCDS;
    return bid < full ? (bid % XCDS) * (nblocks / XCDS) + bid / XCDS : bid;
}
__device__ __forceinline__ void panel_tile(int lid, int tiles_m, int tiles_n, int &tm, int &tn)
{
    constexpr int PANEL = 8;
    const int per_panel = PANEL * tiles_m;
    const int panel = lid / per_panel;
    const int in_panel = lid - panel * per_panel;
    const int width = min(PANEL, tiles_n - panel * PANEL);
    tm = in_panel / width;
    tn = panel * PANEL + in_panel % width;
}
__device__ __forceinline__ void tile_of_block(int bid, int nblocks, int tiles_m, int tiles_n, int &tm,
                                              int &tn)
{
    panel_tile(xcd_logical_id(bid, nblocks), tiles_m, tiles_n, tm, tn);
}

// Expert groups of the grouped products (Appendix A.4): rows of A, or the reduction axis, sorted by expert.
struct GemmGroups {
    const int32_t *ends;  // device memory, `count` non-decreasing row numbers, the last one <= M
    int count;
    int64_t b_group_bytes, bs_group_bytes;
};

// Where the tiles of a problem do not fill the last round over the units, the rest of them (at most `most`) is computed as quarters
// (gemm_staged.h), by a second launch or at the end of the first. units = 0: no such split.
struct GemmTail {
    int units, most;
    // how many of n tiles are computed whole
    __host__ __device__ int first(int n) const
    {
        const int rest = units > 0 ? n % units : 0;
        return n > units && rest <= most ? n - rest : n;
    }
};

// Tile `u` of the tiles of all experts (BM rows each, tiles_n per row of tiles): its expert, that expert's rows [begin, end) and
// the tile's place among the expert's. Ends are clamped to [previous end, M]. u is smaller than grouped_tiles().
struct GroupTile {
    int expert, begin, end, tm, tn;
};
template <int BM> __device__ __forceinline__ int grouped_tiles(const GemmGroups &groups, int M, int tiles_n)
{
    int n = 0;
    for (int e = 0, prev = 0; e < groups.count; ++e) {
        const int end = min(max(groups.ends[e], prev), M);
        n += (end - prev + BM - 1) / BM * tiles_n;
        prev = end;
    }
    return n;
}
template <int BM> __device__ __forceinline__ GroupTile grouped_tile(const GemmGroups &groups, int M, int tiles_n, int u)
{
    GroupTile t = {0, 0, 0, 0, 0};
    int tiles_e = 0;
    for (; t.expert < groups.count; ++t.expert) {
        t.end = min(max(groups.ends[t.expert], t.begin), M);
        tiles_e = (t.end - t.begin + BM - 1) / BM * tiles_n;
        if (u < tiles_e)
            break;
        u -= tiles_e;
        t.begin = t.end;
    }
    panel_tile(xcd_logical_id(u, tiles_e), tiles_e / tiles_n, tiles_n, t.tm, t.tn);
    return t;
}

// Nothing may be scheduled across this point: the instruction order below is the schedule.
#define MXFP8_PIN() __builtin_amdgcn_sched_barrier(0)
// s_waitcnt vmcnt(n), other counters untouched (gfx9 encoding: vmcnt is split over bits 3:0 and 15:14)
#define MXFP8_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// Workgroup barrier without the LDS fence of __syncthreads(): LDS reads issued before it may still be in
// flight afterwards. The persistent kernel uses it where a barrier only publishes DMA-written buffers
// (their arrival is tracked by vmcnt) and nothing that is still being read is handed back for overwriting.
// Where a buffer IS handed back (end of a K step) the reads that can still be in flight are awaited first
// (MXFP8_WAIT_VMCNT_AND_LDS): fragment reads that an already issued MFMA consumed have returned by
// construction, the in-place refills of the A fragments are the only ones left.
#define MXFP8_BARRIER() __builtin_amdgcn_s_barrier()
// s_waitcnt vmcnt(n) lgkmcnt(0): additionally every LDS read of this wavefront has returned
#define MXFP8_WAIT_VMCNT_AND_LDS(n) __builtin_amdgcn_s_waitcnt(0x0070 | ((n) & 15) | (((n) >> 4) << 14))
// Keeps the compiler from moving memory accesses across this point.
#define MXFP8_FENCE() asm volatile("" ::: "memory")

// One K step of one 16x16 output tile. MXFP8: one scaled matrix instruction over 128 k (4 blocks per
// operand row, scale byte 0 of each lane's scale register). BF16: the lane's two 16-byte pieces are k
// 8g..8g+7 and 32+8g..32+8g+7 of the row's 64 values: two 16x16x32 instructions. MXFP4: the lane's two
// 16-byte pieces are scale blocks g and 4+g of the row's 8 (with 4-bit elements a lane holds one whole block
// and its own scale byte applies to it): two scaled instructions over 128 k each; the scale registers carry
// the byte of block g in bits 7:0 and that of block 4+g in bits 15:8.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
template <class Cfg>
__device__ __forceinline__ v4f mma_step(const v8i &first, const v8i &second, v4f acc, int s_first, int s_second)
{
    constexpr int FMT = Cfg::FMT;
    if constexpr (FMT == kFmtFp8) {
        // format fields: 0 = E4M3, 1 = E5M2; the kernels feed B fragments as the first operand, A as the second
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(first, second, acc, Cfg::B_E5M2 ? 1 : 0, Cfg::A_E5M2 ? 1 : 0, 0,
                                                                s_first, 0, s_second);
    } else if constexpr (FMT == kFmtFp4) {
        const v8i f0 = {first[0], first[1], first[2], first[3], 0, 0, 0, 0}, f1 = {first[4], first[5], first[6], first[7], 0, 0, 0, 0};
        const v8i s0 = {second[0], second[1], second[2], second[3], 0, 0, 0, 0}, s1 = {second[4], second[5], second[6], second[7], 0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f0, s0, acc, 4, 4, 0, s_first & 0xFF, 0, s_second & 0xFF);
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f1, s1, acc, 4, 4, 0, (int)((uint32_t)s_first >> 8), 0,
                                                                (int)((uint32_t)s_second >> 8));
    } else {
        const v4i f0 = {first[0], first[1], first[2], first[3]}, f1 = {first[4], first[5], first[6], first[7]};
        const v4i s0 = {second[0], second[1], second[2], second[3]}, s1 = {second[4], second[5], second[6], second[7]};
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, f0), __builtin_bit_cast(v8bf, s0), acc, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, f1), __builtin_bit_cast(v8bf, s1), acc, 0, 0, 0);
    }
}

// Scale register of one fragment from a scale buffer in LDS ([dword][row][4], `rows` tile rows): MXFP8 takes the
// byte of the lane's K block, MXFP4 the bytes of blocks g and 4+g (same position in the two dwords of the row).
template <class Cfg> __device__ __forceinline__ int read_scale(const uint8_t *sbuf, int off, int rows)
{
    if constexpr (Cfg::FMT == kFmtFp4)
        return (int)sbuf[off] | ((int)sbuf[rows * 4 + off] << 8);
    else if constexpr (Cfg::FMT == kFmtFp8)
        return sbuf[off];
    else
        return 0;
}

}  // namespace mxfp8
