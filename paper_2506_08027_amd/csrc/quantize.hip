// MXFP8 quantizer for gfx950: FP32/BF16 -> E4M3 elements + UE8M0 block scales, along rows, along columns, or both from a
// single read of the source (Section 3.2): the grid and its order over the tiles that quantize_tile.h converts.
#include "quantize_tile.h"

namespace mxfp8 {

template <bool BF16, bool ROW, bool COL, bool TILED, int MODE, bool MXSRC = false>
__global__ __launch_bounds__(kQuantThreads) void quantize_kernel(
    const uint8_t *__restrict__ src, int64_t rows, int64_t cols, int64_t ld_bytes,
    uint8_t *__restrict__ q_row, uint8_t *__restrict__ s_row, uint8_t *__restrict__ q_colT,
    uint8_t *__restrict__ s_colT, uint32_t tiles_x, uint32_t ntiles, const uint8_t *__restrict__ src_s)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds_q[COL ? kTile * kTile : 16];
    __shared__ __attribute__((aligned(16))) uint8_t lds_rs[ROW ? kTile * 4 : 16];
    __shared__ __attribute__((aligned(16))) uint8_t lds_cs[COL ? kTile * 4 : 16];
    __shared__ __attribute__((aligned(16))) uint8_t lds_src[MXSRC ? kTile * kTile : 16];
    __shared__ uint32_t lds_src_s[MXSRC ? kTile : 4];
    const QuantLds lds{lds_q, lds_rs, lds_cs, lds_src, lds_src_s};

    // a workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ... (one tile each when the grid has one per tile)
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        // Order of the tiles over the workgroup ids: along the rows of the source, except that a wide tensor (more
        // columns than rows) whose column copy is wanted is walked down its columns, so that the workgroups running
        // side by side append to the same rows of the transposed copy. Measured on an MI355X over six shapes, both
        // source types: 6 % (both copies) to 17 % (column copy only) less time where the rule switches, 5 .. 30 %
        // more wherever it does not.
        const bool walk_down = COL && cols > rows;
        const uint32_t tiles_y = ntiles / tiles_x;
        const uint32_t tile_y = walk_down ? tile % tiles_y : tile / tiles_x, tile_x = walk_down ? tile / tiles_y : tile % tiles_x;
        quantize_tile<BF16, ROW, COL, TILED, MODE, MXSRC>(src, rows, cols, ld_bytes, q_row, s_row, q_colT, s_colT, src_s, tile_y, tile_x,
                                                          (int)threadIdx.x, lds);
        __syncthreads();  // the next tile reuses the staging arrays
    }
}

template <bool BF16, bool TILED, int MODE>
static hipError_t launch_quantize_t(const void *src, int64_t rows, int64_t cols, int64_t ld, int axis,
                                    uint8_t *q_row, uint8_t *s_row, uint8_t *q_colT, uint8_t *s_colT,
                                    hipStream_t stream)
{
    const int64_t tiles_x = (cols + kTile - 1) / kTile;
    const int64_t tiles_y = (rows + kTile - 1) / kTile;
    if (tiles_x * tiles_y > 0x7FFFFFFF)
        return hipErrorInvalidConfiguration;
    // One workgroup per tile, except where a resident grid that walks over the tiles measured faster on an
    // MI355X: the both-axes pass over BF16 sources with 4 workgroups per compute unit (+6 % on [8192 x 4096];
    // FP32 sources and other grid sizes gained nothing).
    int64_t groups = tiles_x * tiles_y;
    if (BF16 && axis == 3) {
        int dev = 0, cus = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess)
            e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess)
            return e;
        if (cus > 0 && groups > 4 * (int64_t)cus)
            groups = 4 * (int64_t)cus;
    }
    dim3 grid((unsigned)groups);
    dim3 block(kQuantThreads);
    const uint8_t *s = static_cast<const uint8_t *>(src);
    const int64_t ldb = ld * (BF16 ? 2 : 4);
    if (axis == 1)
        hipLaunchKernelGGL((quantize_kernel<BF16, true, false, TILED, MODE>), grid, block, 0, stream, s, rows, cols, ldb,
                           q_row, s_row, q_colT, s_colT, (uint32_t)tiles_x, (uint32_t)(tiles_x * tiles_y), static_cast<const uint8_t *>(nullptr));
    else if (axis == 2)
        hipLaunchKernelGGL((quantize_kernel<BF16, false, true, TILED, MODE>), grid, block, 0, stream, s, rows, cols, ldb,
                           q_row, s_row, q_colT, s_colT, (uint32_t)tiles_x, (uint32_t)(tiles_x * tiles_y), static_cast<const uint8_t *>(nullptr));
    else
        hipLaunchKernelGGL((quantize_kernel<BF16, true, true, TILED, MODE>), grid, block, 0, stream, s, rows, cols, ldb,
                           q_row, s_row, q_colT, s_colT, (uint32_t)tiles_x, (uint32_t)(tiles_x * tiles_y), static_cast<const uint8_t *>(nullptr));
    return hipGetLastError();
}

template <int MODE>
static hipError_t launch_quantize_mode(const void *src, bool bf16, int64_t rows, int64_t cols, int64_t ld, int axis,
                                       uint8_t *q_row, uint8_t *s_row, uint8_t *q_colT, uint8_t *s_colT,
                                       bool tiled_scales, hipStream_t stream)
{
    if (tiled_scales)
        return bf16 ? launch_quantize_t<true, true, MODE>(src, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, stream)
                    : launch_quantize_t<false, true, MODE>(src, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, stream);
    return bf16 ? launch_quantize_t<true, false, MODE>(src, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, stream)
                : launch_quantize_t<false, false, MODE>(src, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, stream);
}

// mode: bit 0 = E5M2 elements, bit 1 = OCP v1 scale rule (0 = the recipe)
// Column copy of a tensor derived from its MXFP8 row copy (see quantize_tile, MXSRC).
hipError_t launch_requantize_colwise(const uint8_t *q_row, const uint8_t *s_row, int64_t rows, int64_t cols, uint8_t *q_colT,
                                     uint8_t *s_colT, bool tiled_scales, hipStream_t stream)
{
    const int64_t tiles_x = (cols + kTile - 1) / kTile, tiles_y = (rows + kTile - 1) / kTile;
    if (tiles_x * tiles_y > 0x7FFFFFFF)
        return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(tiles_x * tiles_y)), block(kQuantThreads);
    uint8_t *none = nullptr;
    if (tiled_scales)
        hipLaunchKernelGGL((quantize_kernel<false, false, true, true, 0, true>), grid, block, 0, stream, q_row, rows, cols, cols, none,
                           none, q_colT, s_colT, (uint32_t)tiles_x, (uint32_t)(tiles_x * tiles_y), s_row);
    else
        hipLaunchKernelGGL((quantize_kernel<false, false, true, false, 0, true>), grid, block, 0, stream, q_row, rows, cols, cols, none,
                           none, q_colT, s_colT, (uint32_t)tiles_x, (uint32_t)(tiles_x * tiles_y), s_row);
    return hipGetLastError();
}

hipError_t launch_quantize(const void *src, bool bf16, int64_t rows, int64_t cols, int64_t ld, int axis,
                           uint8_t *q_row, uint8_t *s_row, uint8_t *q_colT, uint8_t *s_colT, bool tiled_scales,
                           int mode, hipStream_t stream)
{
    switch (mode) {
    case 1: return launch_quantize_mode<1>(src, bf16, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, tiled_scales, stream);
    case 2: return launch_quantize_mode<2>(src, bf16, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, tiled_scales, stream);
    case 3: return launch_quantize_mode<3>(src, bf16, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, tiled_scales, stream);
    default: return launch_quantize_mode<0>(src, bf16, rows, cols, ld, axis, q_row, s_row, q_colT, s_colT, tiled_scales, stream);
    }
}

}  // namespace mxfp8
