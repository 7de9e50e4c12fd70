// Sufficient-factor reconstruction fused with the SGD step (Sec. 2.1
// "Sufficient Factor Broadcasting"; Eq. 1, Eq. 2):
//
//   W[m][n] <- W[m][n] - lr * sum_{k<K} U[k][m] * V[k][n]
//
// A dense contraction of depth K = P*B with both operands stored K-major
// (row k of U is u_k, row k of V is v_k), on the matrix cores in 32x32 output
// blocks (64 lanes, 16 fp32 accumulator registers per lane).  By default the
// fp32 products are formed on the 16-bit matrix cores from split operands:
// large layers from two fp16 parts split beforehand, three products per fp32
// product (sf_half.h), the others from three bf16 parts split by the tiles,
// six products (sf_direct.h); the fp32 matrix cores (v_mfma_f32_32x32x2_f32)
// are the alternative the caller can choose, and the register-staged variant
// for very large operands always uses them.
//
// Tiling: a workgroup owns a BM x BN block of W and loops over K in steps of
// BK; each wave owns a WM x WN sub-block (WM/32 x WN/32 MFMA blocks): 128 x
// 128 tiles of 64 x 64, or 64 x 64 tiles of 32 x 32 for small layers.  The
// K-slices U[k0:k0+BK, m0:m0+BM] and V[k0:k0+BK, n0:n0+BN] go straight from
// global memory into LDS with the gfx950 LDS-direct buffer loads (each lane
// moves 16 bytes, a wave instruction fills 1 KB of LDS), two slices in
// flight: the next slice streams in while the matrix cores work on the
// current one, with no register staging and no LDS store instructions.
// Out-of-range operand reads are handled by the buffer resource's range
// check (they read 0), so the K tail needs no branch; reads past the end of a
// row in the last tile column fetch the next row's values, which only feed
// outputs outside W that are never stored.  Inside a slice, 16-byte chunks of
// odd rows are stored with their chunk index XOR 8, so the two half-waves of
// an MFMA operand read (rows k and k+1) hit disjoint LDS banks.
//
// The SGD update is the epilogue: W is read once and written once, straight
// from the accumulators, so the gradient is never materialised, with
// non-temporal accesses that leave the L2 to the operand panels.  On tiles
// that lie wholly inside W the first block of W is loaded before the last K
// step (its latency hides behind that step's MFMAs) and no access carries a
// per-element branch.
//
// Tile order: the hardware hands consecutive workgroups to the 8 XCDs in turn,
// and each XCD has its own L2.  Workgroup ids are remapped so that every XCD
// owns one contiguous run of tiles, walked a group of tile rows at a time, so
// the tiles an XCD runs at the same time share U and V panels in its L2.
//
// Operands whose byte offsets do not fit the 32-bit buffer offsets (K*M or
// K*N of 2^29 elements and more, or rows over 4,194,303 elements) take a
// register-staged variant of the same tile with 64-bit addressing.
//
// Launch forms: one workgroup per tile (a layer, or several layers of one K
// as one grouped tile list), or a spread launch whose few workgroups each
// walk several tiles, for running the rebuild thin beside longer PS work.
#include <algorithm>
#include <atomic>
#include <vector>

#include "common.h"
#include "scratch.h"
#include "sf_direct.h"
#include "sf_half.h"
#include "sf_tile.h"

namespace poseidon {
namespace {

// Tile shapes (workgroup BM x BN, K-slices of BK, wave sub-block WM x WN):
// 128 x 128 tiles when there are at least two per CU, else 64 x 64.
struct Mid {
    static constexpr int BM = 128, BN = 128, BK = 16, WM = 64, WN = 64;
};
struct Small {
    static constexpr int BM = 64, BN = 64, BK = 32, WM = 32, WN = 32;
};
constexpr int64_t MID_TILES_PER_CU = 2;
// 64 x 64 tiles of at most this many per CU (two waves per SIMD), given a
// contraction of at least this depth, take the pipelined split
// (Direct::mma_piped).  With and without it: at two tiles per CU 1000 x 2048
// at K = 1024 34.5 against 36.5 us, K = 256 11.3 and 11.3, K = 96 6.8 and 6.8,
// K = 64 6.0 and 5.9; at one 1000 x 1024 at K = 1024 21.8 and 23.4; at a
// sixteenth 256 x 256 at K = 128 4.7 and 4.9; at three 1500 x 2048 at K = 512
// 29.2 and 28.6, at four 2048 x 2048 36.4 and 35.5.
constexpr int64_t PIPED_TILES_PER_CU = 2;
constexpr int64_t PIPED_MIN_K = 128;

// ---------------------------------------------------------------------------
// Register-staged tile for operands beyond 32-bit offsets: K-slices go global
// -> registers -> LDS (row-padded by 4 floats), double-buffered; 64-bit
// addressing throughout, and W rows too long for 32-bit tile offsets
// (WIDE) take guarded 64-bit accesses in the epilogue.
// ---------------------------------------------------------------------------
constexpr int LDS_PAD = 4;

// Load one BK x (4*COLS4) slice of a K-major operand X (row length ld) into
// registers: group j of this thread covers row g / COLS4 and columns
// 4*(g % COLS4) .. +3 with g = tid + j*THREADS.  Out-of-range rows/columns
// read as 0.  Global loads of several dwords need only 4-byte alignment;
// only a group that runs past the end of its row is read element by element.
template <int NV4, int COLS4, int THREADS>
__device__ inline void load_panel(f4 (&r)[NV4], const float* __restrict__ X, int64_t ld, int64_t rows, int64_t k0,
                                  int64_t c0, int tid)
{
#pragma unroll
    for (int j = 0; j < NV4; ++j) {
        const int g = tid + j * THREADS;
        const int64_t k = k0 + g / COLS4;
        const int64_t c = c0 + 4 * (g % COLS4);
        const float* src = X + k * ld + c;
        const bool kin = k < rows;
        if (kin && c + 3 < ld) {
            r[j] = *reinterpret_cast<const f4u*>(src);
        } else {
            r[j].x = (kin && c + 0 < ld) ? src[0] : 0.f;
            r[j].y = (kin && c + 1 < ld) ? src[1] : 0.f;
            r[j].z = (kin && c + 2 < ld) ? src[2] : 0.f;
            r[j].w = (kin && c + 3 < ld) ? src[3] : 0.f;
        }
    }
}

template <int NV4, int COLS4, int THREADS, int LD>
__device__ inline void store_panel(float* lds, const f4 (&r)[NV4], int tid)
{
#pragma unroll
    for (int j = 0; j < NV4; ++j) {
        const int g = tid + j * THREADS;
        *reinterpret_cast<f4*>(lds + (g / COLS4) * LD + 4 * (g % COLS4)) = r[j];
    }
}

template <int BK, int LDA, int LDB, int TM, int TN>
__device__ inline void mma_staged(f16v (&acc)[TM][TN], const float* a_s, const float* b_s)
{
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
        float a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
            a[i] = a_s[kk * LDA + 32 * i];
#pragma unroll
        for (int j = 0; j < TN; ++j)
            b[j] = b_s[kk * LDB + 32 * j];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
}

template <int BM, int BN, int BK, int WM, int WN, bool WIDE, bool MOM>
__device__ __forceinline__ void sf_tile_staged(float* As, float* Bs, float* __restrict__ W,
                                               const float* __restrict__ U, const float* __restrict__ V, int64_t M,
                                               int64_t N, int64_t K, float lr, int tm, int tn,
                                               float* __restrict__ buf, float mu)
{
    using T = SfTile<BM, BN, BK, WM, WN>;
    constexpr int LDA = BM + LDS_PAD, LDB = BN + LDS_PAD;
    constexpr int SA = BK * LDA, SB = BK * LDB;
    constexpr int A_V4 = BK * BM / 4 / T::THREADS, B_V4 = BK * BN / 4 / T::THREADS;
    static_assert(A_V4 * T::THREADS * 4 == BK * BM && B_V4 * T::THREADS * 4 == BK * BN, "staging");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t m0 = static_cast<int64_t>(tm) * BM;
    const int64_t n0 = static_cast<int64_t>(tn) * BN;
    const int wm = (wave / T::NWN) * WM;
    const int wn = (wave % T::NWN) * WN;
    const int lrow = lane >> 5, lcol = lane & 31;

    f16v acc[T::TM][T::TN];
    zero_acc(acc);
    f4 ra[A_V4], rb[B_V4];
    const int64_t nkt = (K + BK - 1) / BK;
    if (nkt > 0) {
        load_panel<A_V4, BM / 4, T::THREADS>(ra, U, M, K, 0, m0, tid);
        load_panel<B_V4, BN / 4, T::THREADS>(rb, V, N, K, 0, n0, tid);
        store_panel<A_V4, BM / 4, T::THREADS, LDA>(As, ra, tid);
        store_panel<B_V4, BN / 4, T::THREADS, LDB>(Bs, rb, tid);
        __syncthreads();
        const int a_off = lrow * LDA + wm + lcol;
        const int b_off = lrow * LDB + wn + lcol;
        for (int64_t kt = 0; kt < nkt; ++kt) {
            const int cur = static_cast<int>(kt & 1);
            if (kt + 1 < nkt) {
                load_panel<A_V4, BM / 4, T::THREADS>(ra, U, M, K, (kt + 1) * BK, m0, tid);
                load_panel<B_V4, BN / 4, T::THREADS>(rb, V, N, K, (kt + 1) * BK, n0, tid);
            }
            mma_staged<BK, LDA, LDB, T::TM, T::TN>(acc, As + cur * SA + a_off, Bs + cur * SB + b_off);
            if (kt + 1 < nkt) {
                store_panel<A_V4, BM / 4, T::THREADS, LDA>(As + (cur ^ 1) * SA, ra, tid);
                store_panel<B_V4, BN / 4, T::THREADS, LDB>(Bs + (cur ^ 1) * SB, rb, tid);
            }
            __syncthreads();
        }
    }
    if constexpr (!WIDE) {
        const bool interior = (m0 + BM <= M) && (n0 + BN <= N);
        const __amdgpu_buffer_rsrc_t wr = tile_rsrc(W, M, N, m0 * N + n0);
        float wv[16];
        if (!MOM && interior)
            load_w_block(wv, wr, ((wm + 4 * lrow) * static_cast<int>(N) + wn + lcol) * 4, static_cast<int>(N) * 4, 0,
                         W_PRE);
        epilogue<T::TM, T::TN, MOM>(acc, wv, wr, buf, M, N, m0, n0, BM, BN, wm, wn, lrow, lcol, interior, lr, mu);
    } else {
#pragma unroll
        for (int i = 0; i < T::TM; ++i) {
#pragma unroll
            for (int j = 0; j < T::TN; ++j) {
                const int64_t col = n0 + wn + 32 * j + lcol;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t row = m0 + wm + 32 * i + 8 * (r >> 2) + 4 * lrow + (r & 3);
                    if (row < M && col < N) {
                        const int64_t e = row * N + col;
                        if constexpr (MOM) {
                            const float nb = fmaf(mu, buf[e], acc[i][j][r]);
                            buf[e] = nb;
                            W[e] = fmaf(-lr, nb, W[e]);
                        } else {
                            W[e] = fmaf(-lr, acc[i][j][r], W[e]);
                        }
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// How a kernel works one tile: from the operands as they are (fp32 products,
// or bf16 parts split by the tile), loading PRE values of W ahead of the last
// K step (PIPE: with the split pipelined), or from operands split beforehand.
// WAVES: waves per SIMD the kernel
// is compiled for.  Ws: what its launches need of a split operand.
// ---------------------------------------------------------------------------
template <class TL, bool SPLIT, int PRE, bool PIPE = false>
struct DirectProducts {
    static constexpr int BM = TL::BM, BN = TL::BN;
    static constexpr int THREADS = SfTile<BM, BN, TL::BK, TL::WM, TL::WN>::THREADS;
    static constexpr int WAVES = 4;
    struct Ws {
        Ws() = default;
        __host__ __device__ Ws(const SplitWs&) {}
    };
    template <bool MOM>
    static __device__ __forceinline__ void tile(float* W, const float* U, const float* V, int64_t M, int64_t N,
                                                int64_t K, float lr, int tm, int tn, float* buf, float mu, Ws, Ws)
    {
        sf_tile_direct<BM, BN, TL::BK, TL::WM, TL::WN, SPLIT, MOM, PRE, PIPE>(W, U, V, M, N, K, lr, tm, tn, buf, mu);
    }
};

struct HalfProducts {
    static constexpr int BM = HALF_TILE, BN = HALF_TILE;
    static constexpr int THREADS = HALF_THREADS;
    static constexpr int WAVES = 2;
    using Ws = SplitWs;
    template <bool MOM>
    static __device__ __forceinline__ void tile(float* W, const float* U, const float* V, int64_t M, int64_t N,
                                                int64_t K, float lr, int tm, int tn, float* buf, float mu,
                                                const SplitWs& wu, const SplitWs& wv)
    {
        sf_tile_half<MOM>(W, U, V, M, N, K, lr, tm, tn, buf, mu, wu, wv);
    }
};

// ---------------------------------------------------------------------------
// Kernels.
// ---------------------------------------------------------------------------
template <class X, bool MOM>
__global__ __launch_bounds__(X::THREADS) __attribute__((amdgpu_waves_per_eu(X::WAVES, X::WAVES))) void sf_apply_kernel(
    float* __restrict__ W, const float* __restrict__ U, const float* __restrict__ V, int64_t M, int64_t N, int64_t K,
    float lr, int tiles_m, int tiles_n, float* __restrict__ buf, float mu, typename X::Ws wu,
    typename X::Ws wv)
{
    int tm, tn;
    tile_coords<TILE_ROWS>(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    X::template tile<MOM>(W, U, V, M, N, K, lr, tm, tn, buf, mu, wu, wv);
}

// The spread launch: fewer workgroups than tiles (a multiple of 8, so that
// tile t stays on the XCD of workgroup t % 8), each walking the tiles
// grid-stride.  A kernel of its own: the loop makes the compiler keep more
// values live (the fp32 128 x 128 tile spilled 61 VGPRs at the one-tile
// kernel's 128), and a spread launch has few workgroups resident, so it is
// compiled for 2 waves per SIMD (two workgroups per CU).  The barrier keeps a
// wave's first loads of the next tile out of the LDS stage the others may
// still read.
template <class X, bool MOM>
__global__ __launch_bounds__(X::THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void sf_apply_walk_kernel(
    float* __restrict__ W, const float* __restrict__ U, const float* __restrict__ V, int64_t M, int64_t N, int64_t K,
    float lr, int tiles_m, int tiles_n, float* __restrict__ buf, float mu, typename X::Ws wu,
    typename X::Ws wv)
{
    const int tiles = tiles_m * tiles_n;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        if (t != static_cast<int>(blockIdx.x))
            __syncthreads();
        int tm, tn;
        tile_coords<TILE_ROWS>(t, tiles, tiles_m, tiles_n, tm, tn);
        X::template tile<MOM>(W, U, V, M, N, K, lr, tm, tn, buf, mu, wu, wv);
    }
}

template <class TL, bool WIDE, bool MOM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void sf_apply_staged_kernel(
    float* __restrict__ W, const float* __restrict__ U, const float* __restrict__ V, int64_t M, int64_t N, int64_t K,
    float lr, int tiles_m, int tiles_n, float* __restrict__ buf, float mu)
{
    __shared__ float As[2 * TL::BK * (TL::BM + LDS_PAD)];
    __shared__ float Bs[2 * TL::BK * (TL::BN + LDS_PAD)];
    int tm, tn;
    tile_coords<TILE_ROWS>(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    sf_tile_staged<TL::BM, TL::BN, TL::BK, TL::WM, TL::WN, WIDE, MOM>(As, Bs, W, U, V, M, N, K, lr, tm, tn, buf, mu);
}

// ---------------------------------------------------------------------------
// Several layers in one launch (same K): one tile list, so the chip is filled
// by the tiles of the next layer while the last ones of a layer finish,
// instead of every layer ending in a partly idle round.  Layer descriptors
// travel by value in the kernel arguments; the XCD-aware order runs over the
// combined list (layer by layer, in the order given), and inside a layer tile
// rows are walked TILE_ROWS at a time.
// ---------------------------------------------------------------------------
struct SfBatchItem {
    float* W;
    const float* U;
    const float* V;
    int64_t M;
    int64_t N;
    int32_t first_tile;
    int32_t tiles_m;
    int32_t tiles_n;
    int32_t pad;
    SplitWs wu;
    SplitWs wv;
};

struct SfBatchArgs {
    SfBatchItem item[SF_BATCH_MAX];
    int32_t count;
    int32_t total_tiles;
};

template <class X>
__global__ __launch_bounds__(X::THREADS)
__attribute__((amdgpu_waves_per_eu(X::WAVES, X::WAVES))) void sf_apply_batch_kernel(const SfBatchArgs args, int64_t K,
                                                                                  float lr)
{
    const int tiles = args.total_tiles;
    const int q = tiles / NUM_XCD, r = tiles % NUM_XCD;
    const int x = blockIdx.x % NUM_XCD, j = blockIdx.x / NUM_XCD;
    const int t = x * q + (x < r ? x : r) + j;
    int l = 0;
    while (l + 1 < args.count && t >= args.item[l + 1].first_tile)
        ++l;
    const SfBatchItem& it = args.item[l];
    int tm, tn;
    tile_in_list(t - it.first_tile, TILE_ROWS, it.tiles_m, it.tiles_n, tm, tn);
    X::template tile<false>(it.W, it.U, it.V, it.M, it.N, K, lr, tm, tn, nullptr, 0.f, it.wu, it.wv);
}

// True when the LDS-direct tile's 32-bit buffer offsets cover the layer: the
// operand reads (K + BK rows, so the last slice's rows past K still have
// representable offsets) and the W offsets inside one BM-row tile.
bool direct_fits(int64_t M, int64_t N, int64_t K, int BM, int BN, int BK)
{
    constexpr int64_t LIM = 0x7fffffffLL;
    return (K + BK) * M * 4 < LIM && (K + BK) * N * 4 < LIM && (static_cast<int64_t>(BM) * N + BN) * 4 < LIM;
}

// Workgroups of the spread kernel that one CU holds at once (its register
// and LDS needs; cached per instantiation).
template <class X, bool MOM>
int64_t walk_groups_per_cu()
{
    static std::atomic<int> cached{0};
    int n = cached.load(std::memory_order_relaxed);
    if (n > 0)
        return n;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sf_apply_walk_kernel<X, MOM>, X::THREADS, 0) != hipSuccess ||
        n < 1)
        n = 1;
    cached.store(n, std::memory_order_relaxed);
    return n;
}

// A workgroup's rate when few of them walk a layer's tiles beside the PS
// applies (the 1000 x 2048 classifier at K = 1024: 8 tiles of 64 x 64 each
// on 64 workgroups in 0.52 ms, 1.29e11 flop/s), a little under.
constexpr double SPREAD_WG_FLOPS_PER_S = 1.2e11;

// One layer that the LDS-direct and split tiles cover, with X's products
// (ROOM: X without values of W loaded ahead).
template <class X, class ROOM, bool MOM>
hipError_t launch_tiles(float* W, float* buf, const float* U, const float* V, int64_t M, int64_t N, int64_t K,
                        float lr, float mu, double spread_s, bool room, hipStream_t stream, const SplitWs (&ws)[2])
{
    const int64_t tiles_m = (M + X::BM - 1) / X::BM;
    const int64_t tiles_n = (N + X::BN - 1) / X::BN;
    if (tiles_m * tiles_n > INT32_MAX)
        return hipErrorInvalidValue;
    const int t = static_cast<int>(tiles_m * tiles_n), tmi = static_cast<int>(tiles_m),
              tni = static_cast<int>(tiles_n);
    // Spread: as few workgroups (a multiple of 8) as walk the tiles within
    // spread_s at SPREAD_WG_FLOPS_PER_S each -- provided the chip holds them
    // all at once (otherwise the later ones would wait for the first to
    // finish all their tiles).
    if (spread_s > 0.0) {
        const double per = spread_s * SPREAD_WG_FLOPS_PER_S / (2.0 * X::BM * X::BN * static_cast<double>(K));
        if (per >= 2.0) {
            const int64_t p = per < t ? static_cast<int64_t>(per) : t;
            const int64_t g = ((t + p - 1) / p + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
            if (g < t && g <= walk_groups_per_cu<X, MOM>() * device_cu_count()) {
                sf_apply_walk_kernel<X, MOM><<<static_cast<int>(g), X::THREADS, 0, stream>>>(W, U, V, M, N, K, lr,
                                                                                           tmi, tni, buf, mu, ws[0], ws[1]);
                return hipGetLastError();
            }
        }
    }
    if (room)
        sf_apply_kernel<ROOM, MOM><<<t, X::THREADS, 0, stream>>>(W, U, V, M, N, K, lr, tmi, tni, buf, mu, ws[0],
                                                                 ws[1]);
    else
        sf_apply_kernel<X, MOM><<<t, X::THREADS, 0, stream>>>(W, U, V, M, N, K, lr, tmi, tni, buf, mu, ws[0], ws[1]);
    return hipGetLastError();
}

// A layer beyond 32-bit offsets.
template <class TL, bool MOM>
hipError_t launch_staged(float* W, float* buf, const float* U, const float* V, int64_t M, int64_t N, int64_t K,
                         float lr, float mu, hipStream_t stream)
{
    const int64_t tiles_m = (M + TL::BM - 1) / TL::BM;
    const int64_t tiles_n = (N + TL::BN - 1) / TL::BN;
    if (tiles_m * tiles_n > INT32_MAX)
        return hipErrorInvalidValue;
    const int t = static_cast<int>(tiles_m * tiles_n), tmi = static_cast<int>(tiles_m),
              tni = static_cast<int>(tiles_n);
    if ((static_cast<int64_t>(TL::BM) * N + TL::BN) * 4 < 0x7fffffffLL)
        sf_apply_staged_kernel<TL, false, MOM><<<t, 256, 0, stream>>>(W, U, V, M, N, K, lr, tmi, tni, buf, mu);
    else
        sf_apply_staged_kernel<TL, true, MOM><<<t, 256, 0, stream>>>(W, U, V, M, N, K, lr, tmi, tni, buf, mu);
    return hipGetLastError();
}

template <class TL>
int64_t tiles_of(int64_t M, int64_t N)
{
    return ((M + TL::BM - 1) / TL::BM) * ((N + TL::BN - 1) / TL::BN);
}

int64_t panels_of(int64_t n) { return (n + PANEL - 1) / PANEL; }
int64_t round_up(int64_t n, int64_t to) { return (n + to - 1) / to * to; }

// Scratch bytes of one split operand of `len` columns.
struct SplitBytes {
    int64_t planes, exps, flags;
    int64_t total() const { return planes + exps + flags; }
};

SplitBytes split_bytes(int64_t len, int64_t K)
{
    const int64_t groups = (K + GROUP - 1) / GROUP;
    return {panels_of(len) * groups * GROUP_V4 * 16, round_up(panels_of(len) * 4, 256),
            panels_of(len) * round_up(groups, 64)};
}

// Whether a layer's operands are split beforehand (its tiles are 128 x 128
// ones then: at least two per CU).  The pass costs 5-10 us and 8 bytes of
// traffic per factor value, and halves the products.  Measured with and
// without it: 2048 x 2048 tiles' worth at K = 512 (4.3 GFLOP) 32.7 against 36.2
// us, at K = 256 23.3 against 22.1; 4096 x 4096 at K = 128 (4.3 GFLOP) 38.9
// against 40.4, at K = 64 37.5 against 33.2; 8192 x 8192 at K = 64 (8.6 GFLOP)
// 126 against 118, since W's traffic bounds so shallow a product.  A long thin
// layer has as many factor values as outputs: 300 x 25088 at K = 512, M*N/(M+N)
// = 296, 67.9 against 72.8; 64 x 20000 at K = 1024, 64, 53 against 33.
constexpr double PRESPLIT_MIN_FLOPS = 4e9;
constexpr int64_t PRESPLIT_MIN_K = 128, PRESPLIT_MIN_SIDE = 256;

bool presplit_pays(int64_t M, int64_t N, int64_t K)
{
    const double m = static_cast<double>(M), n = static_cast<double>(N);
    return K >= PRESPLIT_MIN_K && 2.0 * m * n * static_cast<double>(K) >= PRESPLIT_MIN_FLOPS &&
           m * n >= PRESPLIT_MIN_SIDE * (m + n);
}

// Splits the operands of `count` layers (at most SF_BATCH_MAX) into scratch:
// ws[2i] is layer i's U, ws[2i+1] its V.  False when the scratch cannot be had
// (nothing is enqueued then).
bool presplit(Scratch& scratch, const SfTensor* t, int32_t count, int64_t K, SplitWs* ws, hipStream_t stream,
              hipError_t& e)
{
    int64_t need = 0;
    for (int32_t i = 0; i < count; ++i)
        need += split_bytes(t[i].M, K).total() + split_bytes(t[i].N, K).total();
    if (!scratch.acquire(static_cast<size_t>(need), stream))
        return false;
    PresplitArgs a{};
    a.K = static_cast<int32_t>(K);
    a.groups = static_cast<int32_t>((K + GROUP - 1) / GROUP);
    a.stride = static_cast<int32_t>(round_up(a.groups, 64));
    a.blocks_per_panel = (a.groups + 4 * PRESPLIT_GROUPS - 1) / (4 * PRESPLIT_GROUPS);
    char* at = static_cast<char*>(scratch.data());
    int32_t blocks = 0;
    for (int32_t i = 0; i < count; ++i)
        for (int k = 0; k < 2; ++k) {
            const int64_t len = k ? t[i].N : t[i].M;
            const SplitBytes b = split_bytes(len, K);
            PresplitItem& it = a.item[a.count++];
            it.X = k ? t[i].V : t[i].U;
            it.len = static_cast<int32_t>(len);
            it.planes = reinterpret_cast<u32x4*>(at);
            it.exps = reinterpret_cast<int*>(at + b.planes);
            it.flags = reinterpret_cast<unsigned char*>(at + b.planes + b.exps);
            at += b.total();
            it.first_block = blocks;
            blocks += static_cast<int32_t>(panels_of(len)) * a.blocks_per_panel;
            ws[2 * i + k] = SplitWs{it.planes, it.exps, it.flags, a.stride};
        }
    sf_presplit_kernel<<<blocks, 256, 0, stream>>>(a);
    e = hipGetLastError();
    return true;
}

template <class TL, bool SPLIT, bool MOM>
hipError_t launch_tl(float* W, float* buf, const float* U, const float* V, int64_t M, int64_t N, int64_t K, float lr,
                     float mu, double spread_s, bool room, hipStream_t stream)
{
    if (!direct_fits(M, N, K, TL::BM, TL::BN, TL::BK))
        return launch_staged<TL, MOM>(W, buf, U, V, M, N, K, lr, mu, stream);
    SplitWs ws[2] = {};
    if constexpr (SPLIT && TL::BM == HALF_TILE) {
        if (presplit_pays(M, N, K)) {
            const SfTensor one{W, U, V, M, N};
            Scratch scratch;
            hipError_t e = hipSuccess;
            if (presplit(scratch, &one, 1, K, ws, stream, e)) {
                if (e != hipSuccess)
                    return e;
                return launch_tiles<HalfProducts, HalfProducts, MOM>(W, buf, U, V, M, N, K, lr, mu, spread_s, false,
                                                                     stream, ws);
            }
        }
    }
    if constexpr (SPLIT && TL::BM == Small::BM) {
        if (spread_s <= 0.0 && !room && K >= PIPED_MIN_K &&
            tiles_of<TL>(M, N) <= PIPED_TILES_PER_CU * device_cu_count()) {
            using X = DirectProducts<TL, true, W_PRE, true>;
            const int tm = static_cast<int>((M + X::BM - 1) / X::BM), tn = static_cast<int>((N + X::BN - 1) / X::BN);
            sf_apply_kernel<X, MOM><<<tm * tn, X::THREADS, 0, stream>>>(W, U, V, M, N, K, lr, tm, tn, buf, mu, ws[0],
                                                                        ws[1]);
            return hipGetLastError();
        }
    }
    // (The momentum epilogue loads no W ahead anyway.)
    using X = DirectProducts<TL, SPLIT, W_PRE>;
    using ROOM = DirectProducts<TL, SPLIT, MOM ? W_PRE : 0>;
    return launch_tiles<X, ROOM, MOM>(W, buf, U, V, M, N, K, lr, mu, spread_s, room, stream, ws);
}

// Tile choice (see Mid, Small).
template <bool SPLIT, bool MOM>
hipError_t launch_sf(float* W, float* buf, const float* U, const float* V, int64_t M, int64_t N, int64_t K, float lr,
                     float mu, double spread_s, bool room, hipStream_t stream)
{
    if (tiles_of<Mid>(M, N) >= MID_TILES_PER_CU * device_cu_count())
        return launch_tl<Mid, SPLIT, MOM>(W, buf, U, V, M, N, K, lr, mu, spread_s, room, stream);
    return launch_tl<Small, SPLIT, MOM>(W, buf, U, V, M, N, K, lr, mu, spread_s, room, stream);
}

template <bool MOM>
hipError_t launch_sf_arith(float* W, float* buf, const float* U, const float* V, int64_t M, int64_t N, int64_t K,
                           float lr, float mu, double spread_s, bool room, hipStream_t stream)
{
    if (sf_arithmetic() == POSEIDON_SF_FP32)
        return launch_sf<false, MOM>(W, buf, U, V, M, N, K, lr, mu, spread_s, room, stream);
    return launch_sf<true, MOM>(W, buf, U, V, M, N, K, lr, mu, spread_s, room, stream);
}

// One grouped launch of at most SF_BATCH_MAX layers (every one covered by the
// 32-bit offsets of X's tile).
template <class X>
hipError_t launch_grouped(const SfTensor* t, int32_t count, int64_t K, float lr, hipStream_t stream, const SplitWs* ws)
{
    SfBatchArgs a{};
    int32_t first = 0;
    for (int32_t g = 0; g < count; ++g) {
        const SfTensor& x = t[g];
        SfBatchItem& it = a.item[a.count++];
        it.W = x.W;
        it.U = x.U;
        it.V = x.V;
        it.M = x.M;
        it.N = x.N;
        if (ws) {
            it.wu = ws[2 * g];
            it.wv = ws[2 * g + 1];
        }
        it.tiles_m = static_cast<int32_t>((x.M + X::BM - 1) / X::BM);
        it.tiles_n = static_cast<int32_t>((x.N + X::BN - 1) / X::BN);
        it.first_tile = first;
        first += it.tiles_m * it.tiles_n;
    }
    a.total_tiles = first;
    sf_apply_batch_kernel<X><<<first, X::THREADS, 0, stream>>>(a, K, lr);
    return hipGetLastError();
}

template <bool SPLIT>
hipError_t launch_one(const SfTensor& x, int64_t K, float lr, bool room, hipStream_t stream)
{
    return launch_sf<SPLIT, false>(x.W, nullptr, x.U, x.V, x.M, x.N, K, lr, 0.f, 0.0, room, stream);
}

// Grouped launch: layers that the 128 x 128 tile covers join one list of such
// tiles when it has at least two per CU; the others, and groups too small to
// fill the chip, take per-layer launches.  With split operands a layer joins
// only when its own launch would take the same tiles and products, so that
// its result does not depend on its company; up to SF_BATCH_MAX such layers
// share one pass that splits their operands, as many as the scratch holds.
template <bool SPLIT>
hipError_t launch_batch(const SfTensor* t, int32_t count, int64_t K, float lr, hipStream_t stream, bool room)
{
    const int64_t want = MID_TILES_PER_CU * device_cu_count();
    std::vector<SfTensor> half, rest;
    int64_t mid = 0;
    for (int32_t i = 0; i < count; ++i) {
        const SfTensor& x = t[i];
        if (x.M == 0 || x.N == 0 || K == 0)
            continue;
        const int64_t tm = tiles_of<Mid>(x.M, x.N);
        const bool fits = direct_fits(x.M, x.N, K, Mid::BM, Mid::BN, Mid::BK);
        if (SPLIT && fits && tm >= want && presplit_pays(x.M, x.N, K)) {
            if (tm <= INT32_MAX / SF_BATCH_MAX) {
                half.push_back(x);
                continue;
            }
        } else if (fits && mid + tm <= INT32_MAX) {
            rest.push_back(x);
            mid += tm;
            continue;
        }
        const hipError_t e = launch_one<SPLIT>(x, K, lr, room, stream);
        if (e != hipSuccess)
            return e;
    }
    if constexpr (SPLIT) {
        for (size_t i = 0; i < half.size();) {
            size_t n = 0;
            int64_t bytes = 0;
            while (i + n < half.size() && n < SF_BATCH_MAX) {
                const SfTensor& x = half[i + n];
                bytes += split_bytes(x.M, K).total() + split_bytes(x.N, K).total();
                if (n > 0 && bytes > static_cast<int64_t>(SCRATCH_LAUNCH_MAX))
                    break;
                ++n;
            }
            SplitWs ws[2 * SF_BATCH_MAX];
            Scratch scratch;
            hipError_t e = hipSuccess;
            if (presplit(scratch, half.data() + i, static_cast<int32_t>(n), K, ws, stream, e)) {
                if (e == hipSuccess)
                    e = launch_grouped<HalfProducts>(half.data() + i, static_cast<int32_t>(n), K, lr, stream, ws);
            } else {
                for (size_t k = 0; k < n && e == hipSuccess; ++k)
                    e = launch_one<SPLIT>(half[i + k], K, lr, room, stream);
            }
            if (e != hipSuccess)
                return e;
            i += n;
        }
    }
    for (size_t i = 0; i < rest.size(); i += SF_BATCH_MAX) {
        const int32_t n = static_cast<int32_t>(std::min<size_t>(SF_BATCH_MAX, rest.size() - i));
        hipError_t e = hipSuccess;
        if (mid < want) {
            for (int32_t k = 0; k < n && e == hipSuccess; ++k)
                e = launch_one<SPLIT>(rest[i + k], K, lr, room, stream);
        } else {
            e = room ? launch_grouped<DirectProducts<Mid, SPLIT, 0>>(rest.data() + i, n, K, lr, stream, nullptr)
                     : launch_grouped<DirectProducts<Mid, SPLIT, W_PRE>>(rest.data() + i, n, K, lr, stream, nullptr);
        }
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

std::atomic<int32_t> g_arithmetic{POSEIDON_SF_BF16X6};

}  // namespace

int32_t sf_arithmetic() { return g_arithmetic.load(std::memory_order_relaxed); }

void set_sf_arithmetic(int32_t a) { g_arithmetic.store(a, std::memory_order_relaxed); }

double sf_seconds(int64_t M, int64_t N, int64_t K)
{
    const double mn = static_cast<double>(M) * static_cast<double>(N);
    const double flops = 2.0 * mn * static_cast<double>(K);
    if (sf_arithmetic() == POSEIDON_SF_FP32)
        return flops / SF_FP32_FLOPS_PER_S;
    if (tiles_of<Mid>(M, N) >= MID_TILES_PER_CU * device_cu_count() && presplit_pays(M, N, K))
        return SF_PRESPLIT_S + std::max(flops / SF_HALF_FLOPS_PER_S, 8.0 * mn / SF_HALF_W_BYTES_PER_S);
    return flops / SF_SPLIT_FLOPS_PER_S;
}

hipError_t launch_sf_apply(float* W, const float* U, const float* V, int64_t M, int64_t N, int64_t K, float lr,
                           hipStream_t stream, double spread_s, bool room)
{
    return launch_sf_arith<false>(W, nullptr, U, V, M, N, K, lr, 0.f, spread_s, room, stream);
}

hipError_t launch_sf_apply_momentum(float* W, float* buf, const float* U, const float* V, int64_t M, int64_t N,
                                    int64_t K, float lr, float mu, hipStream_t stream, double spread_s)
{
    return launch_sf_arith<true>(W, buf, U, V, M, N, K, lr, mu, spread_s, false, stream);
}

hipError_t launch_sf_apply_batch(const SfTensor* t, int32_t count, int64_t K, float lr, hipStream_t stream, bool room)
{
    if (sf_arithmetic() == POSEIDON_SF_FP32)
        return launch_batch<false>(t, count, K, lr, stream, room);
    return launch_batch<true>(t, count, K, lr, stream, room);
}

}  // namespace poseidon
