// The per-group update of the parameter-server apply (Sec. 2.1 "Parameter
// Server"; Sec. 4.1 "KV Store"), shared by every kernel that applies dense
// updates: the single-tensor, batched and KV-store launches.
//
//   s_i = sum_{p<P} G_p[i]   (p increasing, fp32)
//   buf_i = fma(mu, buf_i, s_i);  W_i = fma(-lr, buf_i, W_i)
//
// A thread owns one group of four consecutive elements and issues its shard
// loads (up to PS_CHUNK at a time) before the dependent adds; 16-byte
// accesses, aligned (AL) or at 4-byte alignment, all non-temporal (each array
// is touched once).
#pragma once

#include "common.h"

namespace poseidon {

// Shard loads in flight per step when P is a run-time value, and when a
// compile-time P is larger than this: with all 32 shard loads of P = 32 in
// flight a thread holds 128 VGPRs of them; eight at a time (behind a
// scheduling barrier, so that the compiler cannot hoist them all) the
// Inception-shaped step's batched pass runs at 5.60 instead of 5.47 TB/s and
// the P = 16 launches are unchanged (5.84 TB/s).
constexpr int PS_CHUNK = 8;

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at a 4-byte boundary

__device__ inline f4 fma4(float a, f4 b, f4 c)
{
    return f4{fmaf(a, b.x, c.x), fmaf(a, b.y, c.y), fmaf(a, b.z, c.z), fmaf(a, b.w, c.w)};
}

template <bool AL>
__device__ inline f4 ld4(const float* p)
{
    if constexpr (AL)
        return __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
    else
        return __builtin_nontemporal_load(reinterpret_cast<const f4u*>(p));
}

template <bool AL>
__device__ inline void st4(float* p, f4 v)
{
    if constexpr (AL)
        __builtin_nontemporal_store(v, reinterpret_cast<f4*>(p));
    else
        __builtin_nontemporal_store(v, reinterpret_cast<f4u*>(p));
}

// Where worker p's values of a tensor start: P contiguous shards ...
struct Contiguous {
    const float* G;
    int64_t n;
    __device__ const float* operator()(int p) const { return G + static_cast<int64_t>(p) * n; }
};

// ... or one pointer per worker (the KV store): a whole-tensor update, or a
// message whose values for this range sit `delta` elements further on (bit p
// of msg_mask set).
struct PerWorker {
    const float* const* g;
    uint64_t msg_mask;
    int64_t delta;
    __device__ const float* operator()(int p) const { return g[p] + (((msg_mask >> p) & 1) ? delta : 0); }
};

// The last `rem` (0 to 7) shards, p .. P-1, of NG groups of a run-time P: four,
// two and one of them behind uniform branches, all loaded before the first is
// added, in increasing p.  A launch of a few waves per SIMD is bound by the
// chain of its loads' latencies, and one shard after the other made every one
// of these a latency of its own.
template <bool AL, class Src, int NG>
__device__ inline void add_tail(const Src& src, int P, int p, int rem, const int64_t (&e)[NG], f4 (&s)[NG])
{
    f4 t[7][NG];
    const int p2 = p + (rem & 4);
    if (rem & 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int g = 0; g < NG; ++g)
                t[c][g] = ld4<AL>(src(p + c) + e[g]);
    }
    if (rem & 2) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int g = 0; g < NG; ++g)
                t[4 + c][g] = ld4<AL>(src(p2 + c) + e[g]);
    }
    if (rem & 1) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            t[6][g] = ld4<AL>(src(P - 1) + e[g]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (rem & 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int g = 0; g < NG; ++g)
                s[g] += t[c][g];
    }
    if (rem & 2) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int g = 0; g < NG; ++g)
                s[g] += t[4 + c][g];
    }
    if (rem & 1) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            s[g] += t[6][g];
    }
}

// Sum of the P values of elements e .. e+3, in increasing p (CHAIN: of a
// run-time P, the shards behind the last chunk one after another).
template <int PT, bool AL, bool CHAIN, class Src>
__device__ inline f4 sum4(const Src& src, int P, int64_t e)
{
    if constexpr (PT > PS_CHUNK) {
        f4 s = ld4<AL>(src(0) + e);
#pragma unroll
        for (int p0 = 1; p0 < PT; p0 += PS_CHUNK) {
            f4 g[PS_CHUNK];
#pragma unroll
            for (int c = 0; c < PS_CHUNK; ++c)
                if (p0 + c < PT)
                    g[c] = ld4<AL>(src(p0 + c) + e);
#pragma unroll
            for (int c = 0; c < PS_CHUNK; ++c)
                if (p0 + c < PT)
                    s += g[c];
            __builtin_amdgcn_sched_barrier(0);
        }
        return s;
    } else if constexpr (PT > 0) {
        f4 g[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p)
            g[p] = ld4<AL>(src(p) + e);
        f4 s = g[0];
#pragma unroll
        for (int p = 1; p < PT; ++p)
            s += g[p];
        return s;
    } else {
        const int64_t at[1] = {e};
        f4 s[1] = {ld4<AL>(src(0) + e)};
        int p = 1;
        for (; p + PS_CHUNK <= P; p += PS_CHUNK) {
            f4 g[PS_CHUNK];
#pragma unroll
            for (int c = 0; c < PS_CHUNK; ++c)
                g[c] = ld4<AL>(src(p + c) + e);
#pragma unroll
            for (int c = 0; c < PS_CHUNK; ++c)
                s[0] += g[c];
        }
        if constexpr (CHAIN) {
            for (; p < P; ++p)
                s[0] += ld4<AL>(src(p) + e);
        } else {
            add_tail<AL>(src, P, p, P - p, at, s);
        }
        return s[0];
    }
}

// The update of elements e .. min(e + 4, end) - 1 of one tensor.  (CHAIN for
// the batched pass and the KV store, whose one group per thread leaves waves
// enough: without it the batched pass at P = 7 took 13.9 us for 1.0M values
// where it takes 13.2, and 118 for 15M where it takes 114.)
template <int PT, bool MOM, bool AL, bool CHAIN = true, class Src>
__device__ inline void apply_group(float* __restrict__ W, float* __restrict__ buf, const Src& src, int P, int64_t e,
                                   int64_t end, float lr, float mu)
{
    if (e + 3 < end) {
        const f4 s = sum4<PT, AL, CHAIN>(src, P, e);
        f4 w = ld4<AL>(W + e);
        if constexpr (MOM) {
            const f4 b = fma4(mu, ld4<AL>(buf + e), s);
            st4<AL>(buf + e, b);
            w = fma4(-lr, b, w);
        } else {
            w = fma4(-lr, s, w);
        }
        st4<AL>(W + e, w);
    } else {
        for (int64_t k = e; k < end; ++k) {
            float s = src(0)[k];
            for (int p = 1; p < (PT > 0 ? PT : P); ++p)
                s += src(p)[k];
            float w = W[k];
            if constexpr (MOM) {
                const float b = fmaf(mu, buf[k], s);
                buf[k] = b;
                w = fmaf(-lr, b, w);
            } else {
                w = fmaf(-lr, s, w);
            }
            W[k] = w;
        }
    }
}

// Two groups of one tensor, e and e + PS_PAIR_GAP (64 lanes' groups apart, so
// that a wave's two accesses to each array read 2 KB in a row instead of
// 1 KB; the single-tensor launch): when both are whole their loads are issued
// together, AT_ONCE shards at a time; otherwise, and with AT_ONCE 0, the two
// groups are applied one after the other.  Per element the arithmetic and its order
// are apply_group's, so the results are the same, bitwise.  Single-tensor
// launches of 2,621,440 values at P = 32 ran at 5.97-6.03 TB/s against
// 5.49 with one group per thread, 4,194,304 values at P = 8 at 5.43-5.57
// against 4.85-4.90, and 2,359,296 values at P = 16 measured the same
// (5.45-5.54 against 5.46-5.62).  A run-time P with its two groups together and
// add_tail, against one group after the other and one shard of the tail after
// another, momentum included: 1,179,648 values at P = 7 10.6 against 12.2 us
// and at P = 15 17.2 against 18.7, 1,179,649 at P = 12 14.75 against 16.5 and at
// P = 31 31.0 against 34.7 (4.9 TB/s), 6,000,001 at P = 20 98.9 against 110.4;
// add_tail with the groups one after the other 1-10% slower.  AT_ONCE 0 keeps
// that earlier order (see ps_at_once).
constexpr int64_t PS_PAIR_GAP = 256;
constexpr int PS_PAIR_CHUNK = 4;

template <int PT, bool MOM, bool AL, int AT_ONCE = PS_PAIR_CHUNK, class Src>
__device__ inline void apply_pair(float* __restrict__ W, float* __restrict__ buf, const Src& src, int P, int64_t e,
                                  int64_t end, float lr, float mu)
{
    const int64_t e1 = e + PS_PAIR_GAP;
    if (AT_ONCE > 0 && e1 + 3 < end) {
        const int64_t at[2] = {e, e1};
        constexpr int N = AT_ONCE > 0 ? AT_ONCE : 1;   // (not reached with 0)
        f4 s[2] = {ld4<AL>(src(0) + e), ld4<AL>(src(0) + e1)};
        if constexpr (PT > 0) {
#pragma unroll
            for (int p0 = 1; p0 < PT; p0 += N) {
                f4 a[N], b[N];
#pragma unroll
                for (int c = 0; c < N; ++c)
                    if (p0 + c < PT) {
                        a[c] = ld4<AL>(src(p0 + c) + e);
                        b[c] = ld4<AL>(src(p0 + c) + e1);
                    }
#pragma unroll
                for (int c = 0; c < N; ++c)
                    if (p0 + c < PT) {
                        s[0] += a[c];
                        s[1] += b[c];
                    }
                // one chunk of both groups in registers at a time
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            int p = 1;
            for (; p + N <= P; p += N) {
                f4 a[N], b[N];
#pragma unroll
                for (int c = 0; c < N; ++c) {
                    a[c] = ld4<AL>(src(p + c) + e);
                    b[c] = ld4<AL>(src(p + c) + e1);
                }
#pragma unroll
                for (int c = 0; c < N; ++c) {
                    s[0] += a[c];
                    s[1] += b[c];
                }
            }
            add_tail<AL>(src, P, p, P - p, at, s);
        }
        f4 w0 = ld4<AL>(W + e), w1 = ld4<AL>(W + e1);
        if constexpr (MOM) {
            const f4 b0 = fma4(mu, ld4<AL>(buf + e), s[0]);
            const f4 b1 = fma4(mu, ld4<AL>(buf + e1), s[1]);
            st4<AL>(buf + e, b0);
            st4<AL>(buf + e1, b1);
            w0 = fma4(-lr, b0, w0);
            w1 = fma4(-lr, b1, w1);
        } else {
            w0 = fma4(-lr, s[0], w0);
            w1 = fma4(-lr, s[1], w1);
        }
        st4<AL>(W + e, w0);
        st4<AL>(W + e1, w1);
        return;
    }
    apply_group<PT, MOM, AL, AT_ONCE == 0>(W, buf, src, P, e, end, lr, mu);
    if (e1 < end)
        apply_group<PT, MOM, AL, AT_ONCE == 0>(W, buf, src, P, e1, end, lr, mu);
}

// The shards of both groups that a single-tensor launch of a run-time P loads
// together (AT_ONCE); 0 keeps one group and one shard of the tail after
// another.
//
// 0: tensors with waves enough to hide that latency gain nothing from more
// loads in flight, and where most of P is tail lose by them: with momentum,
// 4,194,304 values at P = 5 24.8 us this way against 25.9, at P = 7 29.6 against
// 31.6, 3,100,000 at P = 15 39.2 against 40.4, 2,359,296 at P = 6 16.5 against
// 16.8 (P = 9 at 4,194,304 41.9 against 38.2 and P = 12 48.3 against 46.8: those
// don't); 1,700,000 at P = 3 10.0 against 9.6, at P = 7 14.5 against 13.7, at P =
// 15 24.1 against 22.7.
//
// PS_PAIR_CHUNK: aligned tensors of more than one workgroup per CU, and beyond
// PS_MANY those with a momentum buffer; else PS_CHUNK.  Up to one workgroup per
// CU a launch is bound by the chain of its loads; beyond, memory serves sixteen
// reads a thread at once worse than eight, worst where the shards lie a power of
// two apart.  One group after another, eight at a time, four: with momentum
// 1,048,576 values at P = 25 19.4, 19.6 and 18.8 us, 2,097,152 at P = 25 47.5,
// 42.2 and 38.7, 8,388,608 at P = 24 171, 176 and 169; without 600,000 at P = 25
// 12.9, 14.1 and 13.4, 1,000,000 at P = 24 19.4, 16.5 and 16.1.  300,000 at P = 25:
// eight 8.0, four 8.6; 4,194,304 at P = 20 without momentum 60.9 against 63.1;
// 600,000 at P = 7, whose shards are all tail with eight, 5.9 against 6.3;
// unaligned tensors are 0-4% slower with four.
constexpr int64_t PS_MANY = int64_t{1} << 21;
inline int ps_at_once(int32_t P, int64_t n, bool aligned, bool momentum, int64_t workgroups, int64_t cus)
{
    if (n > PS_MANY && (P < 8 || (P > 12 && P < 16)))
        return 0;
    return aligned && P > 8 && workgroups > cus && (momentum || n <= PS_MANY) ? PS_PAIR_CHUNK : PS_CHUNK;
}

}  // namespace poseidon
