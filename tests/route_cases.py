"""Problems at which the plain products take each kernel and tile on a 256-unit device, and how a launch shows it.
tests/test_host_model_routes.py holds the launches to it, tests/test_gpu_routes.py runs the problems on the GPU."""

K_STEP = {"fp8": 128, "e5m2": 128, "fp4": 256, "bf16": 64}   # elements of a K step of 128 operand bytes


def launch(call, kernel, bm, bn):
    """(workgroups, LDS bytes) of a launch on 256 units; together they tell the kernels and tiles apart."""
    fmt, M, N, _, _, _, tiled, bound = call
    tiles = -(-M // bm) * -(-N // bn)
    dwords = {"fp4": 2, "bf16": 1}.get(fmt, 1)
    two_buffers = 2 * (bm + bn) * (128 + 4 * dwords)
    if kernel == "one-tile":
        return tiles, two_buffers
    if kernel == "resident":
        return min(tiles, bound or 256), two_buffers + 4 * 4608
    groups = 0 if fmt == "bf16" else (bm + 63) // 64 + (bn + 63) // 64
    scales = 4 * groups * (256 * dwords if tiled else 1024)
    return min(tiles, bound or tiles), max(4 * (bm + bn) * 128 + scales, 4 * 4608)


# format, M, N, K steps, BF16 output, padding of the rows of C (elements), tiled scales, bound on workgroups; kernel, tile
ROUTES = [
    # resident 256-row tiles on ragged problems, more tiles than units
    (("fp8", 5600, 5800, 6, True, 0, True, 0), ("resident", 256, 256)),
    (("fp8", 5600, 5800, 6, False, 0, False, 0), ("resident", 256, 256)),
    (("fp8", 2600, 7000, 5, True, 0, False, 0), ("resident", 256, 192)),
    (("fp8", 2600, 7000, 5, False, 0, True, 0), ("resident", 256, 192)),
    (("fp4", 5600, 5800, 4, True, 0, True, 0), ("resident", 256, 256)),
    (("fp4", 2600, 7000, 5, False, 0, False, 0), ("resident", 256, 192)),
    (("bf16", 5600, 5800, 6, True, 0, False, 0), ("resident", 256, 256)),
    (("bf16", 2600, 7000, 5, False, 0, False, 0), ("resident", 256, 192)),
    # 256x192 tiles on whole problems, MXFP4 and BF16 operands
    (("fp4", 2048, 6144, 16, True, 0, True, 0), ("resident", 256, 192)),
    (("bf16", 2048, 6144, 16, False, 0, False, 0), ("resident", 256, 192)),
    # few K steps and several tiles per workgroup; a bound
    (("fp8", 896, 2688, 4, True, 0, False, 40), ("resident", 128, 128)),
    (("bf16", 1664, 4608, 6, False, 0, False, 0), ("resident", 128, 128)),
    (("fp8", 896, 5504, 11, True, 0, True, 40), ("staged", 128, 128)),      # staged, several tiles per workgroup
    (("fp8", 896, 5504, 12, False, 0, False, 40), ("staged", 128, 128)),
    # staged tiles, row-major E5M2 among them
    (("e5m2", 1000, 2880, 13, True, 0, False, 0), ("staged", 128, 128)),
    (("e5m2", 300, 1000, 9, False, 0, False, 0), ("staged", 32, 64)),
    (("e5m2", 70, 1500, 7, False, 0, False, 0), ("staged", 32, 32)),
    (("fp8", 650, 3000, 9, True, 3, True, 0), ("staged", 128, 128)),
    (("fp8", 1000, 1800, 24, False, 0, False, 0), ("staged", 128, 64)),
    (("fp4", 300, 3100, 9, True, 0, False, 0), ("staged", 64, 64)),
    # two one-tile workgroups on a unit; one-tile workgroups where the rows of C do not start on 16 bytes
    (("fp8", 2254, 2584, 10, True, 0, True, 0), ("one-tile", 128, 128)),
    (("bf16", 2120, 3312, 15, True, 0, False, 0), ("one-tile", 128, 128)),
    (("fp8", 6144, 6921, 5, True, 0, False, 0), ("one-tile", 256, 256)),
    (("fp8", 200, 49152, 8, True, 0, True, 0), ("one-tile", 256, 192)),
]

# M, N, K bytes of an operand row: 256x256 tiles for full rounds on 256 units and a rest of 16 or 32 tiles as quarters, whatever the
# operands and the output (17 x 16, 17 x 16 and 17 x 32 tiles; ragged ones, and one row in the last tiles)
TAIL_SHAPES = [(4352, 4096, 3584), (4290, 4016, 3712), (4097, 8000, 8192)]
