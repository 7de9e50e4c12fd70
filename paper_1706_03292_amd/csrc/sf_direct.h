// SF rebuild tiles fed with LDS-direct loads of the fp32 operands: fp32
// products, or products of bf16 parts that each wave splits in registers.
#pragma once

#include "common.h"
#include "sf_tile.h"

namespace poseidon {
namespace {

template <int BM, int BN, int BK, int WM, int WN>
struct SfTile {
    static constexpr int NWM = BM / WM;
    static constexpr int NWN = BN / WN;
    static constexpr int THREADS = NWM * NWN * 64;
    static constexpr int TM = WM / 32;
    static constexpr int TN = WN / 32;
    static_assert(BM % WM == 0 && BN % WN == 0 && WM % 32 == 0 && WN % 32 == 0, "tile");
    static_assert(BK % 2 == 0, "MFMA depth is 2");
};

// ---------------------------------------------------------------------------
// Split-bf16 products (the default arithmetic of layers too small to split
// their operands beforehand, and of values out of those parts' range).  An
// fp32 value x is the exact
// sum of three bf16 values: h = bf16(x) and m = bf16(x - h), each rounded to
// nearest, and l = x - h - m, which has at most 8 significant bits (bf16
// keeps 8 of fp32's 24 and the same exponent range).  A product x*y is the
// sum of the nine products of the parts; the six kept here (h*h, h*m, m*h,
// h*l, l*h, m*m) are each exact in fp32 and formed on the bf16 matrix cores
// with fp32 accumulation.  The three dropped (m*l, l*m, l*l) are below 2^-23
// of |x*y| together and of either sign.  This is the six-product split of
// Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence
// Datatype For Higher-Precision Computations" (ARITH 2019).
// ---------------------------------------------------------------------------
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float fl2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct Split3 {
    bf8 h, m, l;
};

// Two values rounded to bf16 and packed (the first in the low half).
__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    return __builtin_bit_cast(unsigned, __builtin_convertvector((fl2){a, b}, bf2));
}

// The top halves of two fp32 values packed (a's in the low half): exact for
// values of at most 8 significant bits.
__device__ __forceinline__ unsigned pack_top(float a, float b)
{
    return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, b), __builtin_bit_cast(unsigned, a), 0x07060302u);
}

// x minus half HI of the packed pair p (a bf16's fp32 value is its bits in
// the top half of the word).
template <int HI>
__device__ __forceinline__ float minus_half(float x, unsigned p)
{
    return x - __builtin_bit_cast(float, HI ? (p & 0xffff0000u) : (p << 16));
}

// The parts of x[0..7], two values per conversion.
__device__ __forceinline__ Split3 split3(const float (&x)[8])
{
    u32x4 h, m, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const unsigned hp = pack_bf16(x[2 * q], x[2 * q + 1]);
        const float r0 = minus_half<0>(x[2 * q], hp);
        const float r1 = minus_half<1>(x[2 * q + 1], hp);
        const unsigned mp = pack_bf16(r0, r1);
        h[q] = hp;
        m[q] = mp;
        l[q] = pack_top(minus_half<0>(r0, mp), minus_half<1>(r1, mp));
    }
    return {__builtin_bit_cast(bf8, h), __builtin_bit_cast(bf8, m), __builtin_bit_cast(bf8, l)};
}

// acc[j] += A * B_j over 16 values of K: the six products, the small ones
// first, each over every block of the row before the next.
template <int TN>
__device__ __forceinline__ void split_products(f16v (&acc)[TN], const Split3& a, const Split3 (&b)[TN])
{
    auto each = [&](auto pick_a, auto pick_b) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pick_a(a), pick_b(b[j]), acc[j], 0, 0, 0);
    };
    auto H = [](const Split3& x) { return x.h; };
    auto Mi = [](const Split3& x) { return x.m; };
    auto L = [](const Split3& x) { return x.l; };
    each(Mi, Mi);
    each(H, L);
    each(L, H);
    each(H, Mi);
    each(Mi, H);
    each(H, H);
}

// Chunk (16 bytes) c of slice row k is stored at chunk position c ^ swz(k).
__device__ __forceinline__ constexpr int swz(int k) { return (k & 1) << 3; }

// Wait for every outstanding vector-memory load of this wave (the LDS-direct
// loads included); the workgroup barrier that follows makes every wave's
// loads of the slice visible.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

template <int BM, int BN, int BK, int WM, int WN, bool SPLIT, bool PIPE>
struct Direct {
    using T = SfTile<BM, BN, BK, WM, WN>;
    static constexpr int NT = T::THREADS;
    static_assert(!PIPE || (SPLIT && T::TM * T::TN == 1), "mma_piped");
    struct Parts {
        Split3 a, b;
    };
    template <int S> static __device__ __forceinline__ float* A() { return LdsStage<BK * BM, S, 0>::ptr(); }
    template <int S> static __device__ __forceinline__ float* B() { return LdsStage<BK * BN, S, 1>::ptr(); }

    // One BK x BX slice of a K-major operand into an LDS stage.  Wave
    // instruction q fills LDS chunks 64q .. 64q+63 (row-major, BX/4 chunks a
    // row); its lane l loads global chunk (row g / (BX/4), column chunk
    // (g % (BX/4)) ^ swz(row)) with g = 64q + l.  `rs` addresses the operand
    // from the tile's first column; voffsets are bytes from there, and the
    // resource's size makes every read at or past row K return 0.
    template <int BX>
    static __device__ __forceinline__ void issue_panel(__amdgpu_buffer_rsrc_t rs, float* stage, int ld_bytes, int k0,
                                                       int tid)
    {
        constexpr int CPR = BX / 4;
        constexpr int PER = BK * CPR / NT;
        static_assert(PER * NT == BK * CPR, "slice");
        const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int g0 = (wave + j * (NT / 64)) * 64;
            const int g = g0 + lane;
            const int k = g / CPR;
            const int c = (g % CPR) ^ swz(k);
            const int voff = (k0 + k) * ld_bytes + c * 16;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(stage + g0 * 4), 16, voff, 0, 0, 0);
        }
    }

    template <int S>
    static __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t ur, __amdgpu_buffer_rsrc_t vr, int ldu,
                                                 int ldv, int kt, int tid)
    {
        issue_panel<BM>(ur, A<S>(), ldu, kt * BK, tid);
        issue_panel<BN>(vr, B<S>(), ldv, kt * BK, tid);
    }

    // One BK-deep step of the contraction out of LDS stage S.
    template <int S>
    static __device__ __forceinline__ void mma(f16v (&acc)[T::TM][T::TN], int wm, int wn, int lane)
    {
        if constexpr (SPLIT)
            mma_split<S>(acc, wm, wn, lane);
        else
            mma_f32<S>(acc, wm, wn, lane);
    }

    // Split-bf16 step: 16 values of K per MFMA.  Lane l of an operand holds
    // slot q = 0..7 of its row (column) as K index 2q + l/32, the LDS reads
    // of the fp32 step below, eight at a time; A and B use the same slots.
    template <int S>
    static __device__ __forceinline__ void mma_split(f16v (&acc)[T::TM][T::TN], int wm, int wn, int lane)
    {
        static_assert(BK % 16 == 0, "bf16 MFMA depth is 16");
        const float* a_s = A<S>();
        const float* b_s = B<S>();
        const int lrow = lane >> 5, lcol = lane & 31;
        auto at = [&](const float* s, int ld, int kk, int x) {
            const int k = kk + lrow;
            return s[k * ld + ((((x >> 2) ^ swz(k)) << 2) | (x & 3))];
        };
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            Split3 b[T::TN];
#pragma unroll
            for (int j = 0; j < T::TN; ++j) {
                float x[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    x[q] = at(b_s, BN, kk + 2 * q, wn + 32 * j + lcol);
                b[j] = split3(x);
            }
            // One A block row at a time (its parts and B's stay in registers).
#pragma unroll
            for (int i = 0; i < T::TM; ++i) {
                float x[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    x[q] = at(a_s, BM, kk + 2 * q, wm + 32 * i + lcol);
                split_products<T::TN>(acc[i], split3(x), b);
            }
        }
    }

    // Split-bf16 step of a wave with one block: the slice's values are read at
    // once, and each 16 rows are split while the matrix cores work on the 16
    // before them (`p`; zeros at first), which may be the last slice's.  A wave
    // of one block has one chain of six products and as much splitting as a
    // wave of four has per 24, and small layers have only one or two waves per
    // SIMD: reading, splitting and multiplying followed one another (1000 x
    // 2048 at K = 1024, 35 us without its loads: 12 of them the split, 14 the
    // products).  With the two interleaved 36.5 -> 34.5 us, 1000 x 1024 23.4
    // -> 21.8, 512 x 512 22.5 -> 20.7.  Waves that have three others on their
    // SIMD to overlap with gain nothing.  Same products in the same order.
    static constexpr int VALU_PER_MFMA = 18;   // splitting 16 rows of both: 108 (20, 16, 12 and 9 are slower)

    template <int S>
    static __device__ __forceinline__ void mma_piped(f16v (&acc)[T::TM][T::TN], Parts& p, int wm, int wn, int lane)
    {
        const float* a_s = A<S>();
        const float* b_s = B<S>();
        const int lrow = lane >> 5, lcol = lane & 31;
        auto at = [&](const float* s, int ld, int kk, int x) {
            const int k = kk + lrow;
            return s[k * ld + ((((x >> 2) ^ swz(k)) << 2) | (x & 3))];
        };
        float a[BK / 16][8], b[BK / 16][8];
#pragma unroll
        for (int h = 0; h < BK / 16; ++h)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                a[h][q] = at(a_s, BM, 16 * h + 2 * q, wm + lcol);
                b[h][q] = at(b_s, BN, 16 * h + 2 * q, wn + lcol);
            }
#pragma unroll
        for (int h = 0; h < BK / 16; ++h) {
            mma_parts(acc, p);
            p = {split3(a[h]), split3(b[h])};
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);               // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER_MFMA, 0);   // then VALU
            }
        }
    }

    static __device__ __forceinline__ void mma_parts(f16v (&acc)[T::TM][T::TN], const Parts& p)
    {
        const Split3 b[1] = {p.b};
        split_products<1>(acc[0], p.a, b);
    }

    // fp32 step: the MFMA operands of step kk+2 are read while the matrix
    // cores work on step kk.
    template <int S>
    static __device__ __forceinline__ void mma_f32(f16v (&acc)[T::TM][T::TN], int wm, int wn, int lane)
    {
        const float* a_s = A<S>();
        const float* b_s = B<S>();
        const int lrow = lane >> 5, lcol = lane & 31;
        auto at = [&](const float* s, int ld, int kk, int x) {
            const int k = kk + lrow;
            return s[k * ld + ((((x >> 2) ^ swz(k)) << 2) | (x & 3))];
        };
        float a[2][T::TM], b[2][T::TN];
#pragma unroll
        for (int i = 0; i < T::TM; ++i)
            a[0][i] = at(a_s, BM, 0, wm + 32 * i + lcol);
#pragma unroll
        for (int j = 0; j < T::TN; ++j)
            b[0][j] = at(b_s, BN, 0, wn + 32 * j + lcol);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            const int c = (kk >> 1) & 1;
            if (kk + 2 < BK) {
#pragma unroll
                for (int i = 0; i < T::TM; ++i)
                    a[c ^ 1][i] = at(a_s, BM, kk + 2, wm + 32 * i + lcol);
#pragma unroll
                for (int j = 0; j < T::TN; ++j)
                    b[c ^ 1][j] = at(b_s, BN, kk + 2, wn + 32 * j + lcol);
            }
#pragma unroll
            for (int i = 0; i < T::TM; ++i)
#pragma unroll
                for (int j = 0; j < T::TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][i], b[c][j], acc[i][j], 0, 0, 0);
        }
    }

    // Slice kt (not the last) in stage S: wait until it has landed, then
    // start slice kt+1 into the other stage (free: every wave has passed the
    // barrier after reading it) and multiply.
    template <int S>
    static __device__ __forceinline__ void step(f16v (&acc)[T::TM][T::TN], Parts& p, __amdgpu_buffer_rsrc_t ur,
                                                __amdgpu_buffer_rsrc_t vr, int ldu, int ldv, int kt, int wm, int wn,
                                                int lane, int tid)
    {
        wait_loads();
        __syncthreads();
        issue<S ^ 1>(ur, vr, ldu, ldv, kt + 1, tid);
        // Keep the loads ahead of the multiply: left to itself the scheduler
        // sinks them (they have no register results) to the end of the slice,
        // just before the next step waits for them, and their latency is then
        // hidden only by the other workgroups on the CU.
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PIPE)
            mma_piped<S>(acc, p, wm, wn, lane);
        else
            mma<S>(acc, wm, wn, lane);
    }
};

// One BM x BN tile of W: the whole K loop and the fused update.  Slice kt
// lives in stage (nkt-1-kt) & 1, so the last slice is always in stage 0 and
// the loop body and the final step are each emitted once.  An interior tile
// loads PRE values of W ahead of the last K step.
template <int BM, int BN, int BK, int WM, int WN, bool SPLIT, bool MOM, int PRE = W_PRE, bool PIPE = false>
__device__ __forceinline__ void sf_tile_direct(float* __restrict__ W, const float* __restrict__ U,
                                               const float* __restrict__ V, int64_t M, int64_t N, int64_t K,
                                               float lr, int tm, int tn, float* __restrict__ buf, float mu)
{
    using D = Direct<BM, BN, BK, WM, WN, SPLIT, PIPE>;
    using T = SfTile<BM, BN, BK, WM, WN>;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t m0 = static_cast<int64_t>(tm) * BM;
    const int64_t n0 = static_cast<int64_t>(tn) * BN;
    const int wm = (wave / T::NWN) * WM;
    const int wn = (wave % T::NWN) * WN;
    const int lrow = lane >> 5, lcol = lane & 31;
    const bool interior = (m0 + BM <= M) && (n0 + BN <= N);

    f16v acc[T::TM][T::TN];
    zero_acc(acc);
    const int64_t first = m0 * N + n0;
    const __amdgpu_buffer_rsrc_t wr = tile_rsrc(W, M, N, first);
    const int ni = static_cast<int>(N);
    const int voff = ((wm + 4 * lrow) * ni + wn + lcol) * 4;
    float wv[16];
    typename D::Parts p{};

    const int nkt = static_cast<int>((K + BK - 1) / BK);
    if (nkt > 0) {
        const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(U) + m0, static_cast<short>(0), static_cast<int>((K * M - m0) * 4), BUF_RSRC_WORD3);
        const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(V) + n0, static_cast<short>(0), static_cast<int>((K * N - n0) * 4), BUF_RSRC_WORD3);
        const int ldu = static_cast<int>(M) * 4, ldv = static_cast<int>(N) * 4;
        int kt = 0;
        if ((nkt & 1) == 0) {
            D::template issue<1>(ur, vr, ldu, ldv, 0, tid);
            D::template step<1>(acc, p, ur, vr, ldu, ldv, 0, wm, wn, lane, tid);
            kt = 1;
        } else {
            D::template issue<0>(ur, vr, ldu, ldv, 0, tid);
        }
        for (; kt < nkt - 1; kt += 2) {
            D::template step<0>(acc, p, ur, vr, ldu, ldv, kt, wm, wn, lane, tid);
            D::template step<1>(acc, p, ur, vr, ldu, ldv, kt + 1, wm, wn, lane, tid);
        }
        wait_loads();
        __syncthreads();
        if (!MOM && interior)
            load_w_block(wv, wr, voff, ni * 4, 0, PRE);
        if constexpr (PIPE) {
            D::template mma_piped<0>(acc, p, wm, wn, lane);
            D::mma_parts(acc, p);
        } else {
            D::template mma<0>(acc, wm, wn, lane);
        }
    }
    epilogue<T::TM, T::TN, MOM, PRE>(acc, wv, wr, buf, M, N, m0, n0, BM, BN, wm, wn, lrow, lcol, interior, lr, mu);
}

}  // namespace
}  // namespace poseidon
