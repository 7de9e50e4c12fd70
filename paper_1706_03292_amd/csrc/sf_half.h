// SF rebuild of large layers: both operands are split once into two fp16
// parts by a pass of their own (sf_presplit_kernel), and the tiles form the
// fp32 products from three fp16 products.
//
// What bounds it.  The six bf16 products a tile can form from the raw
// operands (sf_direct.h) already run at the rate the card's matrix cores
// sustain in a large bf16 product (1.2 PFLOP/s; a vendor 8192^3 one 1.24):
// only fewer products make the rebuild faster.  Two fp16 parts hold fp32's 24
// bits in three products where bf16 parts need six, but fp16 has a range of
// 2^40, not 2^254, so every 64-column panel of an operand is scaled by a power
// of two, and rows with a value outside the range are found while splitting
// and take the bf16 products.  Splitting in the tile instead of beforehand was
// slower than the six products' gain (one 128 x 128 tile splits each value as
// often as there are tiles in its row or column, at 22 issue cycles a value:
// 21841 x 4096 at K = 512 in 450 us, with the pass in 302-320, six bf16
// products 490).
#pragma once

#include <type_traits>

#include "common.h"
#include "sf_direct.h"
#include "sf_tile.h"

namespace poseidon {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int PANEL = 64;            // columns of an operand panel
constexpr int GROUP = 16;            // rows of K per group: one MFMA deep
constexpr int GROUP_V4 = 4 * 64;     // 16-byte words of a split group
constexpr int SCALE_ROWS = 8;        // rows, spread over K, whose largest value sets a panel's scale

// ---------------------------------------------------------------------------
// Splitting.  With X = x * 2^(12 - e), e the exponent of the panel's largest
// sampled value, h = fp16(X) and m = fp16((X - h) * 2^12), both to nearest.
// For 2^-13 <= |X| < 2^15 (and for 0) neither part leaves fp16's range or
// loses bits to its subnormals, |X - h| <= 2^-11 of X's binade, and
// X - h - m * 2^-12 is 0 for three values in four and else one unit of fp32's
// last place: the parts are as good as fp32's own rounding, whatever the
// scale.  The products kept are h*h and, in an accumulator of their own, m*h
// and h*m (scaled by 2^12 together); the one left out, m*m * 2^-24, is below
// 2^-22 of the product, of either sign, 2^-24.7 in the mean square.  Measured
// against 64-bit sums, N(0, 1) factors: 1.3e-7 of the raw gradient at K = 256
// and 1.7e-7 at K = 512, six bf16 products 2.4e-7 and 3.4e-7 (a third of the
// additions into the accumulator, so a third of its roundings).
// ---------------------------------------------------------------------------
constexpr float M_SCALE = 4096.f, M_UNSCALE = 1.f / 4096.f;
constexpr int X_TOP = 12;            // the sampled maximum comes to [2^12, 2^13)
constexpr int X_BITS_BELOW = 25;     // 2^-13 is 25 binades below 2^12
constexpr int X_BITS_ABOVE = 3;      // 2^15 is 3 above
// Panels whose largest value has an exponent outside take the bf16 products,
// so that no scaled sum comes near the ends of fp32's own range.
constexpr int E_MIN = -60, E_MAX = 40;
// A group's flags: a value below the range; a value above it, or not finite.
constexpr unsigned BELOW = 1, ABOVE = 0x80;

struct PanelScale {
    int e;
    float s;         // 2^(12 - e)
    unsigned lo;     // 2*bits - 1 of the smallest magnitude in range
    unsigned hi;     // 2*bits of the smallest magnitude above it
};

// From the bits of the largest sampled magnitude.
__device__ __forceinline__ PanelScale panel_scale(int top)
{
    const int e = top == 0 ? 0 : (top >> 23) - 127;
    if (e < E_MIN || e > E_MAX)
        return {0, 1.f, 0u, 0u};          // every value is above the range
    return {e, __builtin_bit_cast(float, (127 + X_TOP - e) << 23),
            (static_cast<unsigned>(127 + e - X_BITS_BELOW) << 24) - 1u,
            static_cast<unsigned>(127 + e + X_BITS_ABOVE) << 24};
}

// (On this chip an fp32 multiply or add issues in half the time of a
// conversion or a mixed-precision FMA, and v_fma_mixlo_f16, which would scale
// and round at once, takes twice that.)
__device__ __forceinline__ void split_half(const float* x, float s, u32x4& h, u32x4& m)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const fl2 X = {x[2 * q] * s, x[2 * q + 1] * s};
        const h2 hp = __builtin_convertvector(X, h2);
        const fl2 r = {__builtin_fmaf(x[2 * q], s, -static_cast<float>(hp[0])) * M_SCALE,
                       __builtin_fmaf(x[2 * q + 1], s, -static_cast<float>(hp[1])) * M_SCALE};
        h[q] = __builtin_bit_cast(unsigned, hp);
        m[q] = __builtin_bit_cast(unsigned, __builtin_convertvector(r, h2));
    }
}

// Split operands: `planes` holds panel after panel, each its groups of 16 rows
// one after another, each group two units of 8 rows, h then m, each 64 columns
// of 8 consecutive rows (16 bytes): 1 KB pieces as an LDS stage holds them and
// as a wave instruction moves them.  Rows past K are 0, columns past the
// operand's edge repeat its last one.  `exps` holds a panel's e, `flags` a byte
// per panel and group.
struct SplitWs {
    const u32x4* planes;
    const int* exps;
    const unsigned char* flags;
    int stride;              // flag bytes per panel (a multiple of 64)
};

struct PresplitItem {
    const float* X;
    u32x4* planes;
    int* exps;
    unsigned char* flags;
    int32_t len;             // columns
    int32_t first_block;
};
constexpr int PRESPLIT_MAX = 2 * SF_BATCH_MAX;
struct PresplitArgs {
    PresplitItem item[PRESPLIT_MAX];
    int32_t count;
    int32_t K;
    int32_t groups;
    int32_t stride;
    int32_t blocks_per_panel;
};

// One wave splits PRESPLIT_GROUPS groups of one panel, a column per lane (256
// bytes of a row per load); it samples the panel's scale itself, so the waves
// need nothing of each other.  Bound by memory on large operands (13.3M
// values, 106 MB read and written, in 22 us: 4.8 TB/s, what a copy reaches)
// and by one memory latency and the launch on small ones (2M values in 5-8
// us).  1, 2 and 4 groups per wave measured the same.
constexpr int PRESPLIT_GROUPS = 2;

__global__ __launch_bounds__(256) void sf_presplit_kernel(const PresplitArgs a)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int l = 0;
    while (l + 1 < a.count && static_cast<int>(blockIdx.x) >= a.item[l + 1].first_block)
        ++l;
    const PresplitItem& it = a.item[l];
    const int b = blockIdx.x - it.first_block;
    const int panel = b / a.blocks_per_panel;
    const int g0 = (b % a.blocks_per_panel * 4 + wave) * PRESPLIT_GROUPS;
    if (g0 >= a.groups)
        return;
    const int first = panel * PANEL;
    const int left = it.len - 1 - first < PANEL - 1 ? it.len - 1 - first : PANEL - 1;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(it.X) + first, static_cast<short>(0), (a.K * it.len - first) * 4, BUF_RSRC_WORD3);
    const int voff = 4 * (lane < left ? lane : left);
    // Row k of this lane's column; rows at and past K repeat the last.
    auto row = [&](int k) {
        const int kk = k < a.K ? k : a.K - 1;
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src, voff, kk * it.len * 4, 0));
    };
    float sample[SCALE_ROWS], raw[PRESPLIT_GROUPS * GROUP];
#pragma unroll
    for (int j = 0; j < SCALE_ROWS; ++j)
        sample[j] = row(static_cast<int>(static_cast<int64_t>(j) * a.K / SCALE_ROWS));
#pragma unroll
    for (int j = 0; j < PRESPLIT_GROUPS * GROUP; ++j)
        raw[j] = row(g0 * GROUP + j);
    float big = 0.f;
#pragma unroll
    for (int j = 0; j < SCALE_ROWS; ++j)
        big = fmaxf(big, fabsf(sample[j]));
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
        big = fmaxf(big, __shfl_xor(big, d));
    const PanelScale ps = panel_scale(__builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, big)));
    if (g0 == 0 && lane == 0)
        it.exps[panel] = ps.e;
#pragma unroll
    for (int q = 0; q < PRESPLIT_GROUPS; ++q) {
        const int g = g0 + q;
        if (g >= a.groups)
            break;
        float* x = raw + q * GROUP;
        if ((g + 1) * GROUP > a.K) {
#pragma unroll
            for (int j = 0; j < GROUP; ++j)
                x[j] = g * GROUP + j < a.K ? x[j] : 0.f;
        }
        // (2*bits drops the sign; a zero wraps to the largest word in mn.)
        unsigned mn = 0xffffffffu, mx = 0;
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            const unsigned t = __builtin_bit_cast(unsigned, x[j]) << 1;
            mn = min(mn, t - 1u);
            mx = max(mx, t);
        }
        const unsigned flag = __any(mx >= ps.hi) ? ABOVE : __any(mn < ps.lo) ? BELOW : 0;
        u32x4* d = it.planes + (static_cast<int64_t>(panel) * a.groups + g) * GROUP_V4 + lane;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            u32x4 h, m;
            split_half(x + 8 * u, ps.s, h, m);
            d[u * 128] = h;
            d[u * 128 + 64] = m;
        }
        if (lane == 0)
            it.flags[static_cast<int64_t>(panel) * a.stride + g] = static_cast<unsigned char>(flag);
    }
}

// ---------------------------------------------------------------------------
// The tile: 128 x 128, four waves of 64 x 64 (2 x 2 MFMA blocks), two
// accumulators per block (128 registers), two workgroups per CU.  A slice is
// one group: its four panels' 16 KB go straight from scratch into LDS, 4 KB a
// wave, in a ring of HALF_STAGES stages.  Four and five stages measured as
// three, three workgroups per CU with 16 KB less scratch in flight each the
// same (and 1.5 times the memory traffic), slices of two groups with two
// stages 5% slower.
// ---------------------------------------------------------------------------
constexpr int HALF_TILE = 128, HALF_THREADS = 256, HALF_STAGES = 3;
constexpr int HALF_PANELS = 4;                            // two of U, two of V
constexpr int HALF_STAGE_V4 = HALF_PANELS * GROUP_V4;

template <int S>
__device__ __forceinline__ u32x4* half_stage()
{
    return reinterpret_cast<u32x4*>(LdsStage<HALF_STAGE_V4 * 4, S, 2>::ptr());
}

template <int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Wait until at most N vector-memory operations of this wave are outstanding
// (loads, the LDS-direct ones included, return in order).
template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N < 64, "counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// The six products of bf16 parts for one group of rows with values out of the
// fp16 range, from the raw operands; the sums join the scaled ones of the
// other groups (unscale: the exponent that takes those back).
__device__ __forceinline__ void bf16_group(f16v (&acc)[2][2], __amdgpu_buffer_rsrc_t ur, __amdgpu_buffer_rsrc_t vr,
                                           int ldu, int ldv, int K, int ucols, int vcols, int unscale, int g, int wm,
                                           int wn, int lrow, int lcol)
{
    // All the group's values first: one memory latency.
    float x[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = (i < 2 ? wm : wn) + 32 * (i & 1) + lcol;
        const int cols = i < 2 ? ucols : vcols;
        const int col = 4 * (c < cols ? c : cols - 1);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = g * GROUP + 8 * lrow + q;
            const int row = (k < K ? k : K - 1) * (i < 2 ? ldu : ldv);
            x[i][q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(i < 2 ? ur : vr, row + col, 0, 0));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if ((g + 1) * GROUP > K) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 8; ++q)
                x[i][q] = g * GROUP + 8 * lrow + q < K ? x[i][q] : 0.f;
    }
    const Split3 b[2] = {split3(x[2]), split3(x[3])};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const Split3 a = split3(x[i]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const Split3 bj[1] = {b[j]};
            f16v c[1];
#pragma unroll
            for (int r = 0; r < 16; ++r)
                c[0][r] = 0.f;
            split_products<1>(c, a, bj);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] += __builtin_ldexpf(c[0][r], -unscale);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

template <bool MOM>
__device__ __forceinline__ void sf_tile_half(float* __restrict__ W, const float* __restrict__ U,
                                             const float* __restrict__ V, int64_t M, int64_t N, int64_t K64, float lr,
                                             int tm, int tn, float* __restrict__ buf, float mu, const SplitWs& wu,
                                             const SplitWs& wv)
{
    constexpr int NS = HALF_STAGES;
    constexpr int PER_WAVE = HALF_STAGE_V4 / 64 / 4;      // 1 KB loads per wave and slice: one panel
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t m0 = static_cast<int64_t>(tm) * HALF_TILE;
    const int64_t n0 = static_cast<int64_t>(tn) * HALF_TILE;
    const int wm = (wave >> 1) * PANEL, wn = (wave & 1) * PANEL;
    const int lrow = lane >> 5, lcol = lane & 31;
    const bool interior = (m0 + HALF_TILE <= M) && (n0 + HALF_TILE <= N);
    const int K = static_cast<int>(K64);
    const int groups = (K + GROUP - 1) / GROUP;

    // The tile's panels (the operand's last one repeated past its edge: it
    // only feeds outputs outside W).
    const int npu = static_cast<int>((M + PANEL - 1) / PANEL), npv = static_cast<int>((N + PANEL - 1) / PANEL);
    auto panel_u = [&](int p) { return 2 * tm + p < npu ? 2 * tm + p : npu - 1; };
    auto panel_v = [&](int p) { return 2 * tn + p < npv ? 2 * tn + p : npv - 1; };

    // Wave w loads panel w of every slice: U's two, then V's.
    const bool isv = wave >= 2;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u32x4*>(isv ? wv.planes : wu.planes) +
            static_cast<int64_t>(isv ? panel_v(wave - 2) : panel_u(wave)) * groups * GROUP_V4,
        static_cast<short>(0), groups * GROUP_V4 * 16, BUF_RSRC_WORD3);
    // (Groups past the last are out of the resource's range and read as 0.)
    auto issue = [&](u32x4* stage, int g) {
#pragma unroll
        for (int q = 0; q < PER_WAVE; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void*)(stage + (wave * PER_WAVE + q) * 64), 16,
                                                     lane * 16 + (g * PER_WAVE + q) * 1024, 0, 0, 0);
    };
    // Slice g lives in stage g % NS; NS-1 slices are in flight.
    static_for<NS - 1>([&](auto q) { issue(half_stage<decltype(q)::value>(), decltype(q)::value); });

    // Groups out of range, over the tile's panels: 16 lanes per panel, four
    // groups a lane.
    int below = 0;
    unsigned above = 0;
    {
        const int p = lane >> 4;
        const unsigned char* f = p < 2 ? wu.flags + static_cast<int64_t>(panel_u(p)) * wu.stride
                                       : wv.flags + static_cast<int64_t>(panel_v(p - 2)) * wv.stride;
        for (int g = 4 * (lane & 15); g < groups; g += 64) {
            unsigned v = *reinterpret_cast<const unsigned*>(f + g);
            if (g + 4 > groups)
                v &= 0xffffffffu >> (8 * (g + 4 - groups));
            above |= v & (ABOVE * 0x01010101u);
            below |= v != 0;
        }
    }
    const bool ragged = __any(below != 0);
    // Values above the range: bf16 products for the whole tile, unscaled.
    const bool wide = __any(above != 0);
    const int pu = panel_u(wave >> 1), pv = panel_v(wave & 1);   // this wave's two
    const int unscale = wide ? 0 : wu.exps[pu] + wv.exps[pv] - 2 * X_TOP;

    f16v acc[2][2], low[2][2];
    zero_acc(acc);
    zero_acc(low);
    // This lane's 16-byte words of its first U and V block in a stage.
    const int a_off = ((wave >> 1) * 4 + 2 * lrow) * 64 + lcol;
    const int b_off = ((2 + (wave & 1)) * 4 + 2 * lrow) * 64 + lcol;
    auto mma = [&](const u32x4* stage) {
        h8 a[2][2], b[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                a[i][p] = __builtin_bit_cast(h8, stage[a_off + p * 64 + 32 * i]);
                b[i][p] = __builtin_bit_cast(h8, stage[b_off + p * 64 + 32 * i]);
            }
        auto each = [&](f16v (&c)[2][2], int p, int q) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i][p], b[j][q], c[i][j], 0, 0, 0);
        };
        each(low, 1, 0);
        each(low, 0, 1);
        each(acc, 0, 0);
    };
    const __amdgpu_buffer_rsrc_t wr = tile_rsrc(W, M, N, m0 * N + n0);
    const int n4 = static_cast<int>(N) * 4;
    const int voff = ((wm + 4 * lrow) * static_cast<int>(N) + wn + lcol) * 4;
    // With a momentum buffer it is read ahead, else W.
    const __amdgpu_buffer_rsrc_t xr = MOM ? tile_rsrc(buf, M, N, m0 * N + n0) : wr;
    float ahead_v[4][16];
    auto load_block = [&](float (&v)[16], __amdgpu_buffer_rsrc_t rs, int c) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            v[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff + 128 * (c % 2),
                                                                                acc_row(c / 2, r) * n4, W_AUX));
    };
    auto store = [&](__amdgpu_buffer_rsrc_t rs, int c, int r, float v) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, voff + 128 * (c % 2),
                                              acc_row(c / 2, r) * n4, W_AUX);
    };
    // Slice g in stage S; NW: loads ahead issued after the slice's own; C >= 0:
    // load block C ahead meanwhile.
    auto step = [&](auto s, auto nw, auto c, int g) {
        constexpr int S = decltype(s)::value, C = decltype(c)::value;
        wait_vm<PER_WAVE * (NS - 2) + decltype(nw)::value>();
        __syncthreads();
        issue(half_stage<(S + NS - 1) % NS>(), g + NS - 1);
        // (The waits count operations in this order, and the loads stay ahead
        // of the multiply.)
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (C >= 0)
            load_block(ahead_v[C], xr, C);
        __builtin_amdgcn_sched_barrier(0);
        mma(half_stage<S>());
    };
    using std::integral_constant;
    constexpr integral_constant<int, -1> none{};
    constexpr integral_constant<int, 0> zero{};
    // An interior tile reads W (or buf) during its first slices, a block per
    // slice, so that memory works while the matrix cores do (4096 x 4096 at K =
    // 256, two rounds of tiles: 47-48 us with it, 55-57 without; during the
    // last four slices instead, 51).
    constexpr int HEAD = 6;
    static_assert(HEAD % NS == 0 && HEAD >= 4 + NS - 1, "the slices whose waits count loads of W");
    const bool ahead = interior && groups >= HEAD && !ragged;
    if (ragged) {
        // Slice after slice, the groups out of range by bf16 products.
        const unsigned char* const fu = wu.flags + static_cast<int64_t>(pu) * wu.stride;
        const unsigned char* const fv = wv.flags + static_cast<int64_t>(pv) * wv.stride;
        const int ucols = static_cast<int>(M - m0 < HALF_TILE ? M - m0 : HALF_TILE);
        const int vcols = static_cast<int>(N - n0 < HALF_TILE ? N - n0 : HALF_TILE);
        const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(U) + m0, static_cast<short>(0), static_cast<int>((K64 * M - m0) * 4), BUF_RSRC_WORD3);
        const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(V) + n0, static_cast<short>(0), static_cast<int>((K64 * N - n0) * 4), BUF_RSRC_WORD3);
        for (int g = 0; g < groups; ++g) {
            wait_vm<0>();
            __syncthreads();
            issue(half_stage<0>(), g);
            wait_vm<0>();
            __syncthreads();
            if (wide || __builtin_amdgcn_readfirstlane(fu[g] | fv[g]))
                bf16_group(acc, ur, vr, static_cast<int>(M) * 4, n4, K, ucols, vcols, unscale, g, wm, wn, lrow, lcol);
            else
                mma(half_stage<0>());
        }
    } else {
        int g = 0;
        if (ahead) {
            static_for<HEAD>([&](auto q) {
                constexpr int k = decltype(q)::value;
                // Blocks of W loaded since slice k's own loads.
                constexpr int from = k - NS + 1 > 0 ? k - NS + 1 : 0, to = k < 4 ? k : 4;
                step(integral_constant<int, k % NS>{}, integral_constant<int, (to > from ? 16 * (to - from) : 0)>{},
                     integral_constant<int, (k < 4 ? k : -1)>{}, k);
            });
            g = HEAD;
        }
        for (; g + NS <= groups; g += NS)
            static_for<NS>([&](auto q) { step(q, zero, none, g + decltype(q)::value); });
        static_for<NS - 1>([&](auto q) {
            if (g + decltype(q)::value < groups)
                step(q, zero, none, g + decltype(q)::value);
        });
    }
    // (The loads into LDS end before the workgroup does.)
    wait_vm<0>();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = __builtin_ldexpf(__builtin_fmaf(low[i][j][r], M_UNSCALE, acc[i][j][r]), unscale);
    if (ahead) {
        if constexpr (MOM) {
            // W goes where the second accumulators were, all its loads at once
            // (against half a block of W and buf at a time, nothing ahead:
            // 4096 x 4096 at K = 512 107 -> 101 us, 21841 x 4096 418 -> 398,
            // 4100 x 5000 at K = 300 178 -> 145).
            float w[4][16];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                load_block(w[c], wr, c);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float nb = fmaf(mu, ahead_v[c][r], acc[c / 2][c % 2][r]);
                    store(xr, c, r, nb);
                    store(wr, c, r, fmaf(-lr, nb, w[c][r]));
                }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    store(wr, c, r, fmaf(-lr, acc[c / 2][c % 2][r], ahead_v[c][r]));
        }
    } else {
        float pre[16];
        epilogue<2, 2, MOM, 0>(acc, pre, wr, buf, M, N, m0, n0, HALF_TILE, HALF_TILE, wm, wn, lrow, lcol, interior, lr,
                               mu);
    }
}

}  // namespace
}  // namespace poseidon
