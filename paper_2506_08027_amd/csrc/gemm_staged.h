// Product kernel for problems that 256x256 tiles cannot spread over the chip: smaller tiles, several K steps in
// flight. Same operands, instruction and order of summation as the kernels of gemm.hip (every output element goes
// through the same sequence of matrix instructions, so the results agree bit for bit).
#pragma once
#include "gemm_device.h"

namespace mxfp8 {

// Tile BM x BN per workgroup of 2 x 2 wavefronts, a ring of four K steps in LDS. One stage holds the A rows, the B rows
// (128 bytes each) and, with tiled scales, one scale dword (two for MXFP4) per row.
template <int BM_, int BN_, int FMT_ = kFmtFp8, bool A_E5M2_ = false, bool B_E5M2_ = false>
struct StagedCfg {
    static constexpr int BM = BM_, BN = BN_, WAVES_M = 2, WAVES_N = 2, STAGES = 4, FMT = FMT_;
    static constexpr bool A_E5M2 = A_E5M2_, B_E5M2 = B_E5M2_;
    static constexpr bool SCALED = FMT_ != kFmtBf16;
    static constexpr int SDW = FMT_ == kFmtFp4 ? 2 : 1;     // scale dwords per operand row and K step
    static constexpr int SBLK = FMT_ == kFmtFp4 ? 16 : 32;  // operand bytes per scale block
    static constexpr int WAVES = WAVES_M * WAVES_N, THREADS = 64 * WAVES;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    static constexpr int TM = WM / 16, TN = WN / 16;
    static constexpr int DATA_BYTES = (BM + BN) * BK;
    static constexpr int LOADS = (BM + BN) / 8 / WAVES;     // 8-row requests per wavefront and stage
    // scale rows are fetched in groups of 64 (the unit of the tiled layout)
    static constexpr int AG = (BM + 63) / 64, BG = (BN + 63) / 64, SGROUPS = SCALED ? (AG + BG) * SDW : 0;
    static constexpr int SREQ = (SGROUPS + WAVES - 1) / WAVES;  // scale requests per wavefront and stage (some are made twice)
    static constexpr int STAGE_SCALE_BYTES = SGROUPS * 256;
    // row-major scales: 16 bytes per row = the dwords of SPG steps, QUADS buffers of them
    static constexpr int SPG = 4 / SDW, QUADS = 4, QUAD_BYTES = SCALED ? (AG + BG) * 1024 : 0;
    static constexpr int L = LOADS + SREQ;  // requests per wavefront and stage
    static constexpr int EPI_BYTES = WAVES * kStageBytes;
    static constexpr int lds_bytes(bool tiled)
    {
        const int ring = STAGES * (DATA_BYTES + (tiled ? STAGE_SCALE_BYTES : 0)) + (tiled ? 0 : QUADS * QUAD_BYTES);
        return ring > EPI_BYTES ? ring : EPI_BYTES;
    }
    static_assert(BM % 16 == 0 && BN % 16 == 0 && WM % 16 == 0 && WN % 16 == 0, "whole matrix instructions");
    static_assert((BM + BN) % (8 * WAVES) == 0 && BM % 8 == 0, "8-row requests spread evenly over the wavefronts");
    // a tile's scale rows are those of AG (BG) groups of 64: its first row is a multiple of 64 or it ends within the group's 64
    // (96 rows from a multiple of 32 on reach into two groups wherever they start)
    static_assert((BM % 64 == 0 || 64 % BM == 0) && (BN % 64 == 0 || 64 % BN == 0 || BN == 96), "a tile's scale rows lie in AG and BG groups");
    static_assert((STAGES - 1) * L < 64, "wait counts");
    static_assert(SPG * QUADS > STAGES + 2 * SPG - 3, "a quad buffer is refilled only after its last step was read");
};

// s_waitcnt for the last steps, where fewer requests are outstanding: all but those of the `newer` youngest K steps
template <int N, int L> __device__ __forceinline__ void wait_tail(int newer)
{
    if (newer >= N)
        MXFP8_WAIT_VMCNT_AND_LDS(N * L);
    else if constexpr (N > 0)
        wait_tail<N - 1, L>(newer);
}

// What bounds it: with 128x128 tiles a K step is 16 matrix instructions per wavefront (512 cycles) against 32 KB of
// direct-to-LDS loads and 64 KB of fragment reads per compute unit, and a load takes one to two microseconds to
// arrive; so what matters is how many K steps are in flight.
//
// One K step kt (fragments of kt are in registers, requests of steps kt+1 .. kt+STAGES-1 are under way):
//   wait until step kt+1 has landed and this wavefront's fragment reads of step kt have returned; barrier: step kt+1
//   is there for every wavefront and the ring slot of step kt is free; matrix instructions of step kt, and between them
//   the fragment reads of step kt+1 (into the other register set) and the requests of step kt+STAGES.
//
// Scales. TILED: one dword per row and step, 64 rows contiguous. Row-major scale bytes of one step lie a whole row
// apart, one cache line per row and request; so one request takes the dwords of four neighbouring positions of 16 rows
// (a quarter of a 64-row group, SPG steps) and every stage brings one quarter (two for MXFP4) of a following group of steps.
// [1000 x 2880 x 5760], 128x128 tiles: 32.3 us with one dword per row and step, 25.2 this way, 22.3 with tiled scales.
//
// TAIL: the tiles are the quarters of the 256x256 tiles that the resident kernel left (GemmTail; tiles_m and tiles_n count those
// tiles), of a plain product, in a launch of their own, or (kTailGrouped) of the row-grouped one, whose number only the device
// knows, at the end of the resident kernel; quarters that lie outside the problem or behind the expert's last row are nothing to
// do. 256-row tiles one of which per unit more than fits leave most units idle for a round: plain [4352 x 4096 x 4096], 272 tiles,
// 74.1 -> 69.2 us (BF16 out, tiled scales), 88.0 -> 78.5 (FP32 out, row-major); the grouped product beside its launch.
enum { kNoTail, kTailPlain, kTailGrouped };
template <class Cfg, bool OUT_BF16, bool TILED, int TAIL = kNoTail>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_staged_kernel(
    const uint8_t *__restrict__ a_q, const uint8_t *__restrict__ a_s, const uint8_t *__restrict__ b_q_all, const uint8_t *__restrict__ b_s_all,
    int M_all, int N, int K, uint8_t *__restrict__ c, int64_t ldc_bytes, int tiles_m, int tiles_n, bool vec_store, GemmTail tail)
{
    static_assert(TAIL == kNoTail || (TAIL == kTailPlain && Cfg::BM == 128 && Cfg::BN == 128), "quarters of 256x256 tiles");
    MXFP8_DYNAMIC_LDS(lds);
    [[maybe_unused]] const GemmGroups groups = {nullptr, 0, 0, 0};
#include "gemm_staged_tiles.h"
}

// The same for the rest of a grouped product, from the resident kernel, in its LDS. Both hold the text itself: the kernel that called a
// function for it kept its registers otherwise and took 2.5 % longer (64x64 and 128x64 tiles, row-major scales).
template <class Cfg, bool OUT_BF16, bool TILED>
__device__ __forceinline__ void staged_grouped_rest(
    uint8_t *lds, const uint8_t *__restrict__ a_q, const uint8_t *__restrict__ a_s, const uint8_t *__restrict__ b_q_all, const uint8_t *__restrict__ b_s_all,
    int M_all, int N, int K, uint8_t *__restrict__ c, int64_t ldc_bytes, int tiles_n, GemmTail tail, const GemmGroups &groups)
{
    static_assert(Cfg::BM == 128 && Cfg::BN == 128, "quarters of 256x256 tiles");
    constexpr int TAIL = kTailGrouped, tiles_m = 0;
    constexpr bool vec_store = true;
#include "gemm_staged_tiles.h"
}

}  // namespace mxfp8
