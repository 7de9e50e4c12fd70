// What every SF rebuild tile shares: the order in which tiles are handed to
// the XCDs, and the fused SGD epilogues that read and write W (and buf)
// straight from the MFMA accumulators.
#pragma once

#include "common.h"

namespace poseidon {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes, 4-byte aligned
typedef __attribute__((address_space(3))) void lds_void;

constexpr int NUM_XCD = 8;    // MI355X: 8 accelerator complex dies, one L2 each

// Buffer resource word 3 for raw (untyped) dword accesses on CDNA.  The raw
// buffer builtins move 32-bit integers: values are bit-cast, never converted.
constexpr int BUF_RSRC_WORD3 = 0x00020000;

// Tile rows an XCD's run walks at a time: 8 of 128 rows (the 64 or 128
// workgroups an XCD runs together then read 8 U and 8 or 16 V panels, the
// fewest for so many tiles).
constexpr int TILE_ROWS = 8;

// Tile t of a layer's list, walked `rows` tile rows at a time.
__device__ inline void tile_in_list(int t, int rows, int tiles_m, int tiles_n, int& tm, int& tn)
{
    const int per_group = rows * tiles_n;
    const int g = t / per_group;
    const int first_m = g * rows;
    const int have = (tiles_m - first_m) < rows ? (tiles_m - first_m) : rows;
    const int in = t - g * per_group;
    tm = first_m + in % have;
    tn = in / have;
}

// Workgroup id -> (tile row, tile column): contiguous runs per XCD, GM tile
// rows at a time inside a run.
template <int GM>
__device__ inline void tile_coords(int bid, int tiles, int tiles_m, int tiles_n, int& tm, int& tn)
{
    const int q = tiles / NUM_XCD, r = tiles % NUM_XCD;
    const int x = bid % NUM_XCD, j = bid / NUM_XCD;
    tile_in_list(x * q + (x < r ? x : r) + j, GM, tiles_m, tiles_n, tm, tn);
}

template <int TM, int TN>
__device__ __forceinline__ void zero_acc(f16v (&acc)[TM][TN])
{
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.f;
}

// ---------------------------------------------------------------------------
// Epilogues.  Accumulator register r of lane l holds block row
// 8*(r/4) + 4*(l/32) + r%4, block column l%32.  `wr` (and `br`) address W
// (buf) from the tile's first element; the byte offsets of a tile fit in 31
// bits (the host checks).
// ---------------------------------------------------------------------------

// Row offset (bytes / n4) of accumulator register r in block row i.
__device__ __forceinline__ constexpr int acc_row(int i, int r) { return 32 * i + 8 * (r >> 2) + (r & 3); }

// Values of W's first MFMA block that an interior tile loads ahead of the last
// K step (as many as the register budget holds without spilling).  Launches
// that leave room for PS waves beside the rebuild load none ahead: 118
// instead of 127 VGPRs, so that a SIMD's four SF waves leave it 32.
constexpr int W_PRE = 10;

// Cache policy of the epilogue's W and buf accesses: non-temporal (the
// buffer instructions' nt bit).  Each value is read and written once, and
// without the hint the 128 KB of W a tile moves through the XCD's L2 evicts
// the U and V panel slices the tiles running beside it still read: the
// VGG19-22K grouped launch fetched 1975 MB from memory with it off and
// 1453 MB with it on (algorithmic 966 MB), and the iteration ran 1.2% faster.
constexpr int W_AUX = 2;

__device__ __forceinline__ void load_w_block(float (&wv)[16], __amdgpu_buffer_rsrc_t wr, int voff, int n4, int r0,
                                             int r1)
{
#pragma unroll
    for (int r = r0; r < r1; ++r)
        wv[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, voff, acc_row(0, r) * n4, W_AUX));
}

// Interior tile: one shared lane offset (voff) and uniform row offsets, one
// MFMA block at a time; the first W_PRE values of block 0 are already in wv.
template <int TM, int TN, int PRE>
__device__ __forceinline__ void epi_interior(const f16v (&acc)[TM][TN], float (&wv)[16], __amdgpu_buffer_rsrc_t wr,
                                             int voff, int n4, float lr)
{
#pragma unroll
    for (int c = 0; c < TM * TN; ++c) {
        const int i = c / TN, j = c % TN;
#pragma unroll
        for (int r = (c == 0 ? PRE : 0); r < 16; ++r)
            wv[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                wr, voff + 128 * j, acc_row(i, r) * n4, W_AUX));
#pragma unroll
        for (int r = 0; r < 16; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, fmaf(-lr, acc[i][j][r], wv[r])), wr,
                                                  voff + 128 * j, acc_row(i, r) * n4, W_AUX);
    }
}

// Ragged edge tile: every element gets its own lane offset; an element outside
// W loads the tile's first element instead (always inside W, value unused) and
// is not stored.
template <int TM, int TN>
__device__ __forceinline__ void epi_edge(const f16v (&acc)[TM][TN], __amdgpu_buffer_rsrc_t wr, int ni, int wm, int wn,
                                         int lrow, int lcol, int rows_left, int cols_left, float lr)
{
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = wn + 32 * j + lcol;
            float ev[16];
            int off[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm + 32 * i + 8 * (r >> 2) + 4 * lrow + (r & 3);
                off[r] = (row < rows_left && col < cols_left) ? (row * ni + col) * 4 : 0;
                ev[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, off[r], 0, W_AUX));
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm + 32 * i + 8 * (r >> 2) + 4 * lrow + (r & 3);
                if (row < rows_left && col < cols_left)
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, fmaf(-lr, acc[i][j][r], ev[r])),
                                                          wr, off[r], 0, W_AUX);
            }
            // One MFMA block at a time: keeps the scheduler from hoisting
            // every block's loads and offsets together.
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Momentum on an edge tile: buf <- mu*buf + dW, W <- W - lr*buf, half an MFMA
// block (8 values per lane) at a time, W and buf loads in flight together,
// then both stores; elements outside W as in epi_edge.
template <int TM, int TN>
__device__ __forceinline__ void epi_momentum(const f16v (&acc)[TM][TN], __amdgpu_buffer_rsrc_t wr,
                                             __amdgpu_buffer_rsrc_t br, int ni, int wm, int wn, int lrow, int lcol,
                                             int rows_left, int cols_left, float lr, float mu)
{
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = wn + 32 * j + lcol;
#pragma unroll
            for (int h = 0; h < 16; h += 8) {
                float wv[8], bv[8];
                int off[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int r = h + q;
                    const int row = wm + 32 * i + 8 * (r >> 2) + 4 * lrow + (r & 3);
                    off[q] = (row < rows_left && col < cols_left) ? (row * ni + col) * 4 : 0;
                    wv[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, off[q], 0, W_AUX));
                    bv[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(br, off[q], 0, W_AUX));
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int r = h + q;
                    const int row = wm + 32 * i + 8 * (r >> 2) + 4 * lrow + (r & 3);
                    if (row < rows_left && col < cols_left) {
                        const float nb = fmaf(mu, bv[q], acc[i][j][r]);
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, nb), br, off[q], 0, W_AUX);
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, fmaf(-lr, nb, wv[q])), wr,
                                                              off[q], 0, W_AUX);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// Momentum on an interior tile: one shared lane offset and uniform row offsets
// for both W and buf, half an MFMA block at a time.
template <int TM, int TN>
__device__ __forceinline__ void epi_momentum_interior(const f16v (&acc)[TM][TN], __amdgpu_buffer_rsrc_t wr,
                                                      __amdgpu_buffer_rsrc_t br, int voff, int n4, float lr, float mu)
{
#pragma unroll
    for (int c = 0; c < TM * TN; ++c) {
        const int i = c / TN, j = c % TN;
#pragma unroll
        for (int h = 0; h < 16; h += 8) {
            float wv[8], bv[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                wv[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                    wr, voff + 128 * j, acc_row(i, h + q) * n4, W_AUX));
                bv[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                    br, voff + 128 * j, acc_row(i, h + q) * n4, W_AUX));
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float nb = fmaf(mu, bv[q], acc[i][j][h + q]);
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, nb), br, voff + 128 * j,
                                                      acc_row(i, h + q) * n4, W_AUX);
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, fmaf(-lr, nb, wv[q])), wr,
                                                      voff + 128 * j, acc_row(i, h + q) * n4, W_AUX);
            }
        }
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(float* base, int64_t M, int64_t N, int64_t first)
{
    const int64_t avail = (M * N - first) * 4;
    return __builtin_amdgcn_make_buffer_rsrc(base + first, static_cast<short>(0),
                                             static_cast<int>(avail < 0x7fffffff ? avail : 0x7fffffff),
                                             BUF_RSRC_WORD3);
}

// The epilogue of one tile for offsets that fit 31 bits.  On an interior
// tile the caller has loaded the first PRE values of block 0 into wv.
template <int TM, int TN, bool MOM, int PRE = W_PRE>
__device__ __forceinline__ void epilogue(const f16v (&acc)[TM][TN], float (&wv)[16], __amdgpu_buffer_rsrc_t wr,
                                         float* __restrict__ buf, int64_t M, int64_t N, int64_t m0, int64_t n0,
                                         int BM, int BN, int wm, int wn, int lrow, int lcol, bool interior,
                                         float lr, float mu)
{
    const int ni = static_cast<int>(N);
    const int rows_left = static_cast<int>(M - m0 < BM ? M - m0 : BM);
    const int cols_left = static_cast<int>(N - n0 < BN ? N - n0 : BN);
    if constexpr (MOM) {
        const __amdgpu_buffer_rsrc_t br = tile_rsrc(buf, M, N, m0 * N + n0);
        if (interior)
            epi_momentum_interior<TM, TN>(acc, wr, br, ((wm + 4 * lrow) * ni + wn + lcol) * 4, ni * 4, lr, mu);
        else
            epi_momentum<TM, TN>(acc, wr, br, ni, wm, wn, lrow, lcol, rows_left, cols_left, lr, mu);
    } else if (interior) {
        epi_interior<TM, TN, PRE>(acc, wv, wr, ((wm + 4 * lrow) * ni + wn + lcol) * 4, ni * 4, lr);
    } else {
        epi_edge<TM, TN>(acc, wr, ni, wm, wn, lrow, lcol, rows_left, cols_left, lr);
    }
}

// Each pipeline stage is an LDS object of its own: the compiler can then tell
// that the in-flight LDS-direct loads into one stage do not alias the LDS
// reads of the other, and does not wait for them before reading.
template <int SIZE, int S, int WHICH>
struct LdsStage {
    static __device__ __forceinline__ float* ptr()
    {
        __shared__ float a[SIZE];
        return a;
    }
};

}  // namespace
}  // namespace poseidon
