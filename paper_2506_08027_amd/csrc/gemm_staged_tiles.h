// The tiles of a workgroup on the staged kernel: text of the functions in gemm_staged.h, which bring the template parameters Cfg,
// OUT_BF16, TILED and TAIL and the names lds, a_q, a_s, b_q_all, b_s_all, M_all, N, K, c, ldc_bytes, tiles_m, tiles_n, vec_store,
// tail and groups.
    constexpr int TM = Cfg::TM, TN = Cfg::TN, S = Cfg::STAGES, SDW = Cfg::SDW;
    constexpr int L = Cfg::L, SPG = Cfg::SPG;
    constexpr int STAGE = Cfg::DATA_BYTES + (TILED ? Cfg::STAGE_SCALE_BYTES : 0);
    constexpr int QUAD_OFF = S * STAGE;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;
    const int r16 = lane & 15, g = lane >> 4;
    const int nkb = K / Cfg::SBLK, KT = K / BK;
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
    const int whole_tiles = TAIL == kTailGrouped ? grouped_tiles<256>(groups, M_all, tiles_n) : tiles_m * tiles_n;
    const int done = TAIL == kNoTail ? 0 : tail.first(whole_tiles);  // tiles computed whole, before
    const int ntiles = TAIL == kNoTail ? whole_tiles : 4 * (whole_tiles - done);

    // fragment addresses inside a stage (see gemm.hip for the swizzle)
    const int a_row = wm * Cfg::WM + r16, b_row = wn * Cfg::WN + r16;
    const int a_off0 = a_row * BK + ((g ^ ((a_row >> 1) & 7)) << 4), a_off1 = a_row * BK + (((4 + g) ^ ((a_row >> 1) & 7)) << 4);
    const int b_off0 = (Cfg::BM + b_row) * BK + ((g ^ ((b_row >> 1) & 7)) << 4), b_off1 = (Cfg::BM + b_row) * BK + (((4 + g) ^ ((b_row >> 1) & 7)) << 4);

    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        int tile_m, tile_n;
        int m0, n0, M = M_all;  // rows from M on are not this tile's
        [[maybe_unused]] const uint8_t *b_q = b_q_all, *b_s = b_s_all;
        if constexpr (TAIL == kNoTail) {
            tile_of_block(tile, ntiles, tiles_m, tiles_n, tile_m, tile_n);
            m0 = tile_m * Cfg::BM;
            n0 = tile_n * Cfg::BN;
        } else {
            int first_row = 0;
            if constexpr (TAIL == kTailGrouped) {
                const GroupTile at = grouped_tile<256>(groups, M_all, tiles_n, done + (tile >> 2));
                tile_m = at.tm;
                tile_n = at.tn;
                first_row = at.begin;
                M = at.end;
                b_q += at.expert * groups.b_group_bytes;
                b_s += at.expert * groups.bs_group_bytes;
            } else {
                tile_of_block(done + (tile >> 2), whole_tiles, tiles_m, tiles_n, tile_m, tile_n);
            }
            m0 = first_row + tile_m * 256 + (tile >> 1 & 1) * 128;
            n0 = tile_n * 256 + (tile & 1) * 128;
            if (m0 >= M || n0 >= N)
                continue;
        }

        // ---- requests: 8-row group i of this wavefront, counted over the A rows and then the B rows of the tile
        const int ld_r = lane >> 3, ld_c = lane & 7;
        const uint8_t *src[Cfg::LOADS];
        uint32_t goff[Cfg::LOADS];
#pragma unroll
        for (int i = 0; i < Cfg::LOADS; ++i) {
            const int grp = wave * Cfg::LOADS + i;  // wavefront-uniform
            const bool is_a = grp < Cfg::BM / 8;
            const int row = (is_a ? grp : grp - Cfg::BM / 8) * 8 + ld_r;
            src[i] = is_a ? a_q + (int64_t)m0 * K : b_q + (int64_t)n0 * K;
            // ragged tiles re-read the last valid row
            goff[i] = (uint32_t)min(row, (is_a ? M - m0 : N - n0) - 1) * (uint32_t)K + (ld_c ^ ((row >> 1) & 7)) * 16;
        }
        // scale request j: 64-row group sidx / SDW; scale dword (tiled) or quarter (row-major) sidx % SDW of it
        const uint8_t *ssrc[Cfg::SREQ + 1];
        int sidx[Cfg::SREQ + 1], srow[Cfg::SREQ + 1], slast[Cfg::SREQ + 1];
#pragma unroll
        for (int j = 0; j < Cfg::SREQ; ++j) {
            const int idx = (wave + j * Cfg::WAVES) % (Cfg::SCALED ? Cfg::SGROUPS : 1);  // wavefront-uniform
            sidx[j] = idx;
            const int grp = idx / SDW, dw = idx % SDW;
            const bool is_a = grp < Cfg::AG;
            const int g64 = is_a ? grp : grp - Cfg::AG, first = is_a ? m0 : n0, rows = is_a ? M : N;
            const uint8_t *s = is_a ? a_s : b_s;
            if constexpr (TILED) {
                ssrc[j] = s + (int64_t)min(first / 64 + g64, (rows + 63) / 64 - 1) * KT * (256 * SDW) + dw * 256;
            } else {
                ssrc[j] = s + (int64_t)first * nkb;
                srow[j] = g64 * 64 + dw * 16 + (lane >> 2);
                slast[j] = rows - first - 1;
            }
        }
        // quarter q (of a group whose steps start at first_step) of scale request j's rows
        auto issue_quarter = [&](int j, int first_step, int q) __attribute__((always_inline)) {
            const int dword = min(first_step * SDW + (lane & 3), KT * SDW - 1);  // past the end of the row: its last one again
            const uint32_t off = (uint32_t)min(srow[j] + q * 16, slast[j]) * (uint32_t)nkb + dword * 4;
            dma_load<4>(ssrc[j], off, lds_base + QUAD_OFF + (first_step / SPG % Cfg::QUADS) * Cfg::QUAD_BYTES + (sidx[j] / SDW) * 1024 +
                                          (sidx[j] % SDW + q) * 256);
        };
        // slot t of the requests of K step kt into ring slot `slot`
        auto issue = [&](int t, int kt, int slot) __attribute__((always_inline)) {
            const uint32_t stage = lds_base + slot * STAGE;
            if (t < Cfg::LOADS) {
                dma_load<16>(src[t] + (int64_t)kt * BK, goff[t], stage + (wave * Cfg::LOADS + t) * 1024);
            } else if constexpr (TILED) {
                const int j = t - Cfg::LOADS;
                dma_load<4>(ssrc[j] + (int64_t)kt * (256 * SDW), lane * 4, stage + Cfg::DATA_BYTES + sidx[j] * 256);
            } else {
                // the last quarter of the group of steps G goes out with step SPG * G, its first SPG - 1 steps earlier
                const int ahead = kt + SPG - 1;
                issue_quarter(t - Cfg::LOADS, ahead / SPG * SPG, ahead % SPG * SDW);
            }
        };

        const int sa_row = (TILED ? m0 & 63 : 0) + a_row, sb_row = (TILED ? n0 & 63 : 0) + b_row;
        v8i fa[2][TM], fb[2][TN];
        int sa[2][TM], sb[2][TN];
        // piece p of the fragments of K step kt: 16 bytes of every lane; with the first half of a fragment its scale byte
        constexpr int PIECES = 2 * (TM + TN);
        auto read_piece = [&](int p, int kt, int slot, int set) __attribute__((always_inline)) {
            const uint8_t *stage = lds + slot * STAGE;
            auto scale = [&](int row, int group0) __attribute__((always_inline)) {
                // tiled: [group][dword][64 rows][4], row-major: [group][64 rows][4 dwords][4]
                if constexpr (Cfg::SCALED) {
                    const uint8_t *q = TILED ? stage + Cfg::DATA_BYTES + (group0 + (row >> 6)) * (256 * SDW) + (row & 63) * 4 + g
                                             : lds + QUAD_OFF + (kt / SPG % Cfg::QUADS) * Cfg::QUAD_BYTES + group0 * 1024 + row * 16 +
                                                   (kt % SPG) * (4 * SDW) + g;
                    constexpr int NEXT = TILED ? 256 : 4;  // from one scale dword of a step to the next
                    return SDW == 2 ? (int)q[0] | ((int)q[NEXT * (SDW - 1)] << 8) : (int)q[0];
                } else {
                    return 0;
                }
            };
            const int f = p >> 1, half = p & 1;  // compile-time after unrolling
            const bool is_b = f < TN;
            const int t = is_b ? f : f - TN;
            const v4i v = *reinterpret_cast<const v4i *>(stage + (is_b ? (half ? b_off1 : b_off0) : (half ? a_off1 : a_off0)) + t * 2048);
            v8i &dst = is_b ? fb[set][is_b ? t : 0] : fa[set][is_b ? 0 : t];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                dst[half * 4 + e] = v[e];
            if (half == 0) {
                if (is_b)
                    sb[set][t] = scale(sb_row + t * 16, Cfg::AG);
                else
                    sa[set][t] = scale(sa_row + t * 16, 0);
            }
        };

        v4f acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

        // ---- prologue: the first S steps, before them the scales of the first group of steps
        if constexpr (!TILED && Cfg::SCALED) {
#pragma unroll
            for (int q = 0; q < 4 - SDW; q += SDW)
#pragma unroll
                for (int j = 0; j < Cfg::SREQ; ++j)
                    issue_quarter(j, 0, q);
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int t = 0; t < L; ++t)
                issue(t, s, s);
        }
        MXFP8_WAIT_VMCNT_AND_LDS((S - 1) * L);
        MXFP8_BARRIER();
        MXFP8_FENCE();

        // K step kt with its fragments in register set `set`. `left` (compile-time): steps after this one, up to S.
        int slot = 0;  // ring slot of step kt
        auto step = [&](int kt, int set, int left) __attribute__((always_inline)) {
            const int next = slot + 1 == S ? 0 : slot + 1;
            if (left > 0) {
                // younger than step kt+1: steps kt+2 .. kt+S-1, as far as there are any
                if (left >= S)
                    MXFP8_WAIT_VMCNT_AND_LDS((S - 2) * L);
                else
                    wait_tail<S - 2, L>(left - 1);
                MXFP8_BARRIER();
                MXFP8_FENCE();
            }
            MXFP8_PIN();
#pragma unroll
            for (int m = 0; m < TM * TN; ++m) {
                const int i = m % TM, j = m / TM;
                acc[i][j] = mma_step<Cfg>(fb[set][j], fa[set][i], acc[i][j], sb[set][j], sa[set][i]);
                MXFP8_PIN();
                if (left > 0) {
#pragma unroll
                    for (int p = m * PIECES / (TM * TN); p < (m + 1) * PIECES / (TM * TN); ++p)
                        read_piece(p, kt + 1, next, set ^ 1);
                }
                if (left >= S) {
#pragma unroll
                    for (int t = m * L / (TM * TN); t < (m + 1) * L / (TM * TN); ++t)
                        issue(t, kt + S, slot);
                }
                MXFP8_PIN();
            }
            slot = next;
        };
        // Straight-line bodies: KT - S steps that fetch, an odd one first (so that the last S start with register set 0),
        // then the last S. Branches inside a step, or two bodies that meet again, make the compiler move all accumulators
        // between registers (128 moves a step of 16 matrix instructions were seen).
        int kt = 0;
        if ((KT - S) & 1) {
#pragma unroll
            for (int p = 0; p < PIECES; ++p)
                read_piece(p, 0, 0, 1);
            step(0, 1, S);
            kt = 1;
        } else {
#pragma unroll
            for (int p = 0; p < PIECES; ++p)
                read_piece(p, 0, 0, 0);
        }
        for (; kt < KT - S; kt += 2) {
            step(kt, 0, S);
            step(kt + 1, 1, S);
        }
#pragma unroll
        for (int t = 0; t < S; ++t)
            step(kt + t, t & 1, S - 1 - t);

        // ---- epilogue: 16-row groups through a wavefront-private LDS area (the ring is done with), whole rows out
        constexpr int ESZ = OUT_BF16 ? 2 : 4;
        MXFP8_FENCE();
        __syncthreads();
        const int mw = m0 + wm * Cfg::WM, nw = n0 + wn * Cfg::WN;  // first row and column of this wavefront
        if (vec_store) {
            constexpr int ROWB = Cfg::WN * ESZ, PITCH = ROWB + 32;
            static_assert(16 * PITCH <= kStageBytes, "staging area");
            constexpr int CHUNKS = ROWB / 16;  // 16-byte pieces per row
            uint8_t *area = lds + wave * kStageBytes;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const v4f v = acc[i][j];
                    uint8_t *dst = area + r16 * PITCH + (j * 16 + 4 * g) * ESZ;
                    if constexpr (OUT_BF16) {
                        v2bf p0 = {(__bf16)v[0], (__bf16)v[1]}, p1 = {(__bf16)v[2], (__bf16)v[3]};
                        *reinterpret_cast<uint2 *>(dst) = make_uint2(__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1));
                    } else {
                        *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                    }
                }
                __builtin_amdgcn_wave_barrier();  // the reads below see the other lanes' writes (LDS serves a wavefront in order)
#pragma unroll
                for (int t = 0; t < (16 * CHUNKS + 63) / 64; ++t) {
                    const int piece = t * 64 + lane, row = piece / CHUNKS, colb = (piece % CHUNKS) * 16;
                    const int m = mw + i * 16 + row, n = nw + colb / ESZ;
                    if ((16 * CHUNKS % 64 == 0 || piece < 16 * CHUNKS) && m < M && n < N) {
                        const uint4 v = *reinterpret_cast<const uint4 *>(area + row * PITCH + colb);
                        uint8_t *out = c + (int64_t)m * ldc_bytes + (int64_t)n * ESZ;
                        if (n + 16 / ESZ <= N) {
                            *reinterpret_cast<uint4 *>(out) = v;
                        } else {  // the row ends inside this piece
                            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                            for (int e = 0; e < 16 / ESZ; ++e)
                                if (n + e < N) {
                                    if constexpr (OUT_BF16)
                                        *reinterpret_cast<uint16_t *>(out + e * 2) = (uint16_t)(w[e / 2] >> (16 * (e & 1)));
                                    else
                                        *reinterpret_cast<uint32_t *>(out + e * 4) = w[e];
                                }
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();  // (the next row group overwrites the area after these reads)
            }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int m = mw + i * 16 + r16;
                if (m >= M)
                    continue;
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int n = nw + j * 16 + 4 * g + e;
                        if (n < N) {
                            if constexpr (OUT_BF16)
                                *reinterpret_cast<__bf16 *>(c + (int64_t)m * ldc_bytes + (int64_t)n * 2) = (__bf16)acc[i][j][e];
                            else
                                *reinterpret_cast<float *>(c + (int64_t)m * ldc_bytes + (int64_t)n * 4) = acc[i][j][e];
                        }
                    }
            }
        }
        if (tile + (int)gridDim.x < ntiles)
            __syncthreads();  // the next tile's requests go where the rows were staged
    }
