// fp32 tile GEMM for fp32 problems (the small validation layer) on the fp32 matrix cores: up to 128 x 64 outputs per
// workgroup.  Same contract as the bf16 kernel: the result is left in an LDS C tile (fp32 here).
//
// What bounds it: few tiles (a layer of 256 tokens has 64 to 256 of them), so one tile's latency is the phase's time.
// The four wavefronts therefore split the REDUCTION and not the tile: wavefront w takes the 8-index pieces w, w + 4, ...
// of it for all rows and columns, which shares no operand between wavefronts, so operands go from memory straight into the
// registers the MFMA reads, several pieces ahead, with no LDS and no barrier in the loop; and a tile of few rows costs
// only the 32-row blocks it has (ROWS), with all four wavefronts still at work.  Interleaved pieces make the four
// wavefronts read the same 128-byte line of a row together.  The partial sums meet once, through LDS, at the end.
// (The loop before this one staged 16 indices at a time through LDS with nothing in flight and multiplied on the vector
// ALU, whose FMA rate without packed instructions is half the matrix cores'.)
// Whole layer, that loop -> this one: 256 tokens on 8 experts of 512 x 1024 358 -> 118 us; 1 token on 2 of 16 experts of
// 1024 x 2048 592 -> 87; 64 tokens on 4 of 6144 x 4096 2921 -> 359; 4000 rows on 4 of 512 x 1024 685 -> 298.  Error against
// 64 bits (2-norm, staging) 8.3e-7 -> 4.2e-7 and 2.4e-6 -> 1.2e-6 on the first and third: four shorter sums.
#pragma once
#include "common.hpp"
#include "gemm_bf16.hpp"

namespace moe {

// Most parts of a GEMM2 tile, see g2_join: all of a sum's parts are in flight at once.  6 / 8 parts, us: 128 tokens x 2 of 4 experts of 128 x 2048
// 71.5 / 69.3, of 512 x 2048 85.9 / 85.3, 64 x 2 of 4 of 512 x 4096 92.1 / 90.6: what more could give is less than that.
constexpr int kG2MaxParts = 8;
// Most tiles a layer that cuts them can have, whatever its load: it bounds the parts' sums in the workspace (33 MB) and their counters, a
// cache line each, that every call clears.  Layers beyond it stay whole, which costs some of them time, whole / 2 parts, us: 300 tokens x 2 of 16
// experts of 512 x 1024 (160 tiles at most) 100.5 / 97.5, 400 x 2 of 8 of 1024 x 2048 (224) 198.9 / 179.2; 128 x 1 of 16 of 512 x 512 (136) 68.6 / 70.5.
constexpr int kG2SplitTiles = 128;

struct TileF32 {
    static constexpr int BM = 128, BN = 64;
    static constexpr int BN_NARROW = 32;               // GEMM1 tiles of a layer that has too few of 64 columns (see make_plan)
    static constexpr int C_STRIDE = BN * 4 + 16;       // bytes per C-tile row
    static constexpr int C_BYTES = BM * C_STRIDE;
    // partial sums: each wavefront's for the other three, [dest][3][block of 32 x 32][lane] of 16 bytes
    static constexpr int X_BYTES = 4 * 3 * (BM / 32) * (BN / 32) * 64 * 16;
    static constexpr int SMEM_MAIN = C_BYTES + X_BYTES;
};

// Operands of one piece of 8 reduction indices: lanes 0..31 hold the indices 0..3 of it, lanes 32..63 the indices 4..7
// (MFMA j multiplies index j of both halves).  Column c of a lane is CB * (lane % 32) + c, so that CB = 2 columns are one
// 8-byte load.
template <bool GATED, int ROWS, int CB>
struct PieceF32 {
    float4 a[ROWS];
    float b[GATED ? 2 : 1][4][CB];
};

// Adds the four wavefronts' partial sums of ROWS x CB blocks and leaves a quarter of every block with each wavefront: in
// out[] are the outputs (row lane % 32, block index 8 * wave + 4 * (lane / 32) + 0..3) of every block.  All threads.
template <int ROWS, int CB>
__device__ __forceinline__ void exchange_f32(const f32x16_t (&acc)[ROWS][CB], f32x4_t (&out)[ROWS][CB], char *xbuf, int wave,
                                             int lane) {
    constexpr int NB = ROWS * CB;
    f32x4_t *X = (f32x4_t *)xbuf;
#pragma unroll
    for (int dst = 0; dst < 4; ++dst) {
        const int from = wave < dst ? wave : wave - 1;
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const f32x16_t &v = acc[r][c];
                const f32x4_t q = {v[4 * dst], v[4 * dst + 1], v[4 * dst + 2], v[4 * dst + 3]};
                out[r][c] = dst == 0 || dst == wave ? q : out[r][c];
                if (dst != wave) X[((dst * 3 + from) * NB + r * CB + c) * 64 + lane] = q;
            }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i) out[r][c] += X[((wave * 3 + i) * NB + r * CB + c) * 64 + lane];
}

template <bool GATED, int ROWS, int CB, class RowPtr, class Hook>
__device__ __forceinline__ void gemm_rows_f32(RowPtr rowptr, const float *B0, const float *B1, int ldb, int ncols, int K,
                                              char *smem, Hook while_loading) {
    using C = TileF32;
    // pieces in flight per wavefront: what the registers beside the sums hold (in the forms of 3 and 4 row blocks not all of it:
    // the compiler reports 42 spilled vector registers for the fp32 megakernel, and around the exchange sums go to scratch)
    constexpr int DEPTH = ROWS <= 2 ? 8 : 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int col = min(l32 * CB, ncols - CB);  // (columns past the tile's repeat its last ones and are not stored)
    const int n = (K / 8 - wave + 3) / 4;       // pieces of this wavefront

    const float *arow[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) arow[r] = rowptr(r * 32 + l32) + half * 4;
    const u32 bofs = (u32)(half * 4) * (u32)ldb + (u32)col;  // (below 2^32: four rows of one expert's matrix)

    f32x16_t g[ROWS][CB], u[GATED ? ROWS : 1][CB];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                g[r][c][i] = 0.f;
                if (GATED) u[r][c][i] = 0.f;
            }

    while_loading();  // (first: values that are loaded across it end up copied, and a copy waits for its load)
    PieceF32<GATED, ROWS, CB> s[DEPTH];
    auto load = [&](PieceF32<GATED, ROWS, CB> &p, int i) __attribute__((always_inline)) {
        const int k0 = (4 * min(i, n - 1) + wave) * 8;  // (pieces past the end are the last one again, and not used)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) p.a[r] = *(const float4 *)(arow[r] + k0);
#pragma unroll
        for (int m = 0; m < (GATED ? 2 : 1); ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float *b = (m ? B1 : B0) + (size_t)(k0 + j) * ldb;
                if constexpr (CB == 2) {
                    const float2 v = *(const float2 *)(b + bofs);
                    p.b[m][j][0] = v.x, p.b[m][j][1] = v.y;
                } else {
                    p.b[m][j][0] = b[bofs];
                }
            }
    };
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            load(s[i], i);
            __builtin_amdgcn_sched_barrier(0);  // (pieces are waited for in this order)
        }
    }
    for (int i0 = 0; i0 < n; i0 += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            if (i0 + i < n) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        const float av = j == 0 ? s[i].a[r].x : j == 1 ? s[i].a[r].y : j == 2 ? s[i].a[r].z : s[i].a[r].w;
#pragma unroll
                        for (int c = 0; c < CB; ++c) {
                            g[r][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(s[i].b[0][j][c], av, g[r][c], 0, 0, 0);
                            if (GATED)
                                u[r][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(s[i].b[GATED ? 1 : 0][j][c], av, u[r][c], 0, 0, 0);
                        }
                    }
            }
            load(s[i], i0 + i + DEPTH);  // (also past the end: the number of loads in flight is then known at every wait)
            __builtin_amdgcn_sched_barrier(0);  // (a load that sank to its use would leave nothing in flight)
        }
    }

    char *xbuf = smem + C::C_BYTES;
    f32x4_t o[ROWS][CB];
    exchange_f32<ROWS, CB>(g, o, xbuf, wave, lane);
    if constexpr (GATED) {
        f32x4_t v[ROWS][CB];
        __syncthreads();
        exchange_f32<ROWS, CB>(u, v, xbuf, wave, lane);
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float x = o[r][c][i];
                    o[r][c][i] = x / (1.0f + expf(-x)) * v[r][c][i];
                }
            }
    }
    const int i0 = 8 * wave + 4 * half;  // this lane's outputs within a block
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        char *row = smem + (r * 32 + l32) * C::C_STRIDE + i0 * CB * 4;
        if constexpr (CB == 2) {
            const f32x4_t p = o[r][0], q = o[r][1];
            *(f32x4_t *)row = f32x4_t{p[0], q[0], p[1], q[1]};
            *(f32x4_t *)(row + 16) = f32x4_t{p[2], q[2], p[3], q[3]};
        } else {
            *(f32x4_t *)row = o[r][0];
        }
    }
    __syncthreads();
}

// nrows: rows of the tile that exist (1..BM); ncols: columns that exist (a multiple of 16, at most BN)
template <bool GATED, class RowPtr, class Hook>
__device__ __forceinline__ void gemm_tile_f32(RowPtr rowptr, const float *B0, const float *B1, int ldb, int ncols, int nrows,
                                              int K, char *smem, Hook while_loading) {
    const bool narrow = GATED && ncols <= 32;
    switch ((nrows + 31) / 32 + (narrow ? 4 : 0)) {
        case 1: return gemm_rows_f32<GATED, 1, 2>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        case 2: return gemm_rows_f32<GATED, 2, 2>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        case 3: return gemm_rows_f32<GATED, 3, 2>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        case 4: return gemm_rows_f32<GATED, 4, 2>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        case 5: if constexpr (GATED) return gemm_rows_f32<GATED, 1, 1>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        case 6: if constexpr (GATED) return gemm_rows_f32<GATED, 2, 1>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        case 7: if constexpr (GATED) return gemm_rows_f32<GATED, 3, 1>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
        default: if constexpr (GATED) return gemm_rows_f32<GATED, 4, 1>(rowptr, B0, B1, ldb, ncols, K, smem, while_loading);
    }
}

}  // namespace moe
