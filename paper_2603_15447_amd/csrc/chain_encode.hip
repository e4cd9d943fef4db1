// Zig-zag encoder of C0 piecewise chains (Sec. 2.1, Eq. 2, Fig. 2): the free
// texels of a chain of N segments are fixed by x_0 = M_0 and x_k + x_{k+1} =
// 2 M_k, an alternating prefix sum over the middle points, evaluated here as
// an FP64 block scan (per-block sums, a scan of those, then one pass that
// scans each block's own columns and writes them): every texel is one FP32
// rounding of an FP64 prefix sum, where an FP32 recurrence x_{k+1} = 2 M_k -
// x_k would let the rounding error grow with k.
#include "common.h"

namespace bzi {
namespace {

// The encoder works on "channels": a quadratic chain has DIM channels (one
// per coordinate); a cubic chain (Sec. 2.1, two zig-zag layers stacked front
// to back) has 2*DIM, layer l of coordinate c being channel l*DIM + c.  Both
// layers share the on-path texels A_k = P_3k; their middle points satisfy
// 2 E0_k = 3 P_3k+1 - P_3k and 2 E1_k = 3 P_3k+2 - P_3k+3 (exact in FP64),
// so that the depth lerp of the two layers is the cubic (P_3k .. P_3k+3).
//
// Element e_k = (-1)^(k+1) * 2 M_k of the alternating sum: the free texels are
// x_k = (-1)^k y_k with y_k = M_0 + sum_{j<k} e_j, which is x_{k+1} = 2M_k - x_k.
//
// Both passes are bound by memory (the chain in, the grid out), so all their
// global traffic is contiguous: a block stages the rows of its columns (ROWS
// rows of DIM floats per column, one more row for a cubic's last segment) in
// LDS, every thread scans kEncPerThread consecutive columns there, puts the
// free texels in place of the middle points, and the block writes its part of
// the grid in order.  A thread's columns take an odd number of LDS words, so
// that the 64 lanes of a wave, all at the same place of their own run, meet
// different banks.  At 2^20 3D segments the passes take 7 us (25 MB in), 5
// and 12 us (25 MB in, 25 out).  (Threads that read and wrote their columns in
// global memory, a column pitch of 2*DIM floats apart, took 18, 8 and 85 us;
// with an LDS index computed per float instead of per four, the last pass was
// bound by its index arithmetic and took 18.)
constexpr int kEncPerThread = 4;

template <int DIM, int ROWS, int NT>
struct EncGeom {
    static constexpr int NCH = DIM * (ROWS - 1);
    static constexpr int COLS = NT * kEncPerThread;         // columns per block
    static constexpr int RUN = kEncPerThread * ROWS * DIM;  // floats of a thread's columns in the chain,
    static constexpr int OUT = kEncPerThread * 2 * NCH;     // and in the grid
    static constexpr int N = COLS * ROWS * DIM + (ROWS == 3 ? DIM : 0);  // floats staged
    static constexpr int LDS = NT * ((RUN > OUT ? RUN : OUT) | 1) + (ROWS == 3 ? DIM : 0);
    static constexpr int WAVES = NT / 64;
};

// LDS word of float f, threads' runs of R floats (a multiple of 4, so four
// floats from a multiple of 4 on lie together) an odd number of words apart.
template <int R>
__device__ __forceinline__ int enc_at(int f) { return f + f / R; }

typedef float enc_f4 __attribute__((ext_vector_type(4), aligned(4)));

// Rows of the block's columns [col0, col0 + COLS), zero past the chain's end.
template <int DIM, int ROWS, int NT>
__device__ __forceinline__ void enc_stage(const float *__restrict__ chain, int64_t n_seg, int64_t col0, float *lds) {
    using G = EncGeom<DIM, ROWS, NT>;
    const int64_t first = col0 * ROWS * DIM, total = (n_seg * ROWS + 1) * DIM;
    const float *__restrict__ src = chain + first;
    const int avail = static_cast<int>(min(static_cast<int64_t>(G::N), total - first));
    // all loads first: their latency passes once
    constexpr int IT = (G::N + 4 * NT - 1) / (4 * NT);
    float v[IT][4] = {};
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int f = 4 * (threadIdx.x + i * NT);
        if (f + 4 <= avail) {
            const enc_f4 x = *reinterpret_cast<const enc_f4 *>(src + f);
            v[i][0] = x[0], v[i][1] = x[1], v[i][2] = x[2], v[i][3] = x[3];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (f + e < avail) v[i][e] = src[f + e];
        }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int f = 4 * (threadIdx.x + i * NT), at = enc_at<G::RUN>(f);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (f + e < G::N) lds[at + e] = v[i][e];
    }
}

// 2 M_k of channel ch (an array of column k's rows, then the next column's end point).
template <int DIM, int ROWS, typename P>
__device__ __forceinline__ double enc_twice_mid(const P &row, int ch) {
    if constexpr (ROWS == 2) return 2.0 * static_cast<double>(row(DIM + ch));
    const int layer = ch >= DIM, c = ch - layer * DIM;
    const double a = row(layer ? 3 * DIM + c : c), b = row(layer ? 2 * DIM + c : DIM + c);
    return 3.0 * b - a;
}

// The elements of this thread's columns, from LDS.
template <int DIM, int ROWS, int NT>
__device__ __forceinline__ void enc_elems(const float *lds, int64_t n_seg, int64_t col0,
                                          double (&ev)[kEncPerThread][EncGeom<DIM, ROWS, NT>::NCH]) {
    using G = EncGeom<DIM, ROWS, NT>;
    const int64_t k0 = col0 + threadIdx.x * kEncPerThread;
#pragma unroll
    for (int i = 0; i < kEncPerThread; ++i) {
        // (a last column's successor is the next thread's first)
        const float *own = lds + threadIdx.x * (G::RUN | 1) + i * ROWS * DIM;
        auto row = [&](int j) { return own[j + (i * ROWS * DIM + j >= G::RUN ? 1 : 0)]; };
#pragma unroll
        for (int ch = 0; ch < G::NCH; ++ch) {
            const double m2 = enc_twice_mid<DIM, ROWS>(row, ch);
            // k0 is a multiple of 4: column k0 + i is odd when i is
            ev[i][ch] = k0 + i < n_seg ? ((i & 1) ? m2 : -m2) : 0.0;
        }
    }
}

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// A block's sum (later: the sum before the block) waits in the first column of
// the block's own part of the grid, NCH doubles in exactly one column: only
// that block reads it in the last pass, before it writes the column, so the
// encoder needs no workspace.  (hipMallocAsync and hipFreeAsync of a small one
// cost 20 us of host time per call, more than all passes at 2^18 segments.)
struct EncInGrid {
    static constexpr bool kInPlace = false;
    using In = const float *__restrict__;
    using Out = float *__restrict__;
};

// A quadratic chain encoded in place (grid == chain) has no such column, and its
// own first column is gone when the last blocks come to start from M_0: the sums
// wait in a workspace, the block's own behind each other, and M_0 behind them.
struct EncInPlace {
    static constexpr bool kInPlace = true;
    using In = const float *;
    using Out = float *;
    float *ws;  // nullptr: g_enc_scratch
    int64_t nb;
};

// Workspace of chains encoded in place without an allocation: as many doubles as
// the longest of them takes.
constexpr int64_t kEncScratchDoubles = int64_t(1) << 18;
__device__ double g_enc_scratch[kEncScratchDoubles + kMaxDim];

// Place of block b's sum (b = nb in place: of M_0).
template <int NCH>
__device__ __forceinline__ float *enc_place(EncInGrid, float *grid, int64_t cols, int64_t b) { return grid + b * cols * 2 * NCH; }
template <int NCH>
__device__ __forceinline__ float *enc_place(EncInPlace at, float *, int64_t, int64_t b) {
    return (at.ws ? at.ws : reinterpret_cast<float *>(g_enc_scratch)) + b * 2 * NCH;
}

__device__ __forceinline__ void enc_put(float *p, int ch, double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    p[2 * ch] = __uint_as_float(static_cast<uint32_t>(u));
    p[2 * ch + 1] = __uint_as_float(static_cast<uint32_t>(u >> 32));
}
__device__ __forceinline__ double enc_get(const float *p, int ch) {
    return __builtin_bit_cast(double, __float_as_uint(p[2 * ch]) | static_cast<uint64_t>(__float_as_uint(p[2 * ch + 1])) << 32);
}

template <int DIM, int ROWS, int NT, typename S>
__global__ __launch_bounds__(NT) void k_enc_partials(const float *__restrict__ chain, int64_t n_seg, float *__restrict__ grid,
                                                     S sums) {
    using G = EncGeom<DIM, ROWS, NT>;
    __shared__ float lds[G::LDS];
    __shared__ double wsum[G::WAVES][G::NCH];
    const int64_t col0 = static_cast<int64_t>(blockIdx.x) * G::COLS;
    enc_stage<DIM, ROWS, NT>(chain, n_seg, col0, lds);
    __syncthreads();
    double ev[kEncPerThread][G::NCH];
    enc_elems<DIM, ROWS, NT>(lds, n_seg, col0, ev);
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int ch = 0; ch < G::NCH; ++ch) {
        const double s = wave_sum64((ev[0][ch] + ev[1][ch]) + (ev[2][ch] + ev[3][ch]));
        if ((threadIdx.x & 63) == 0) wsum[wave][ch] = s;
    }
    __syncthreads();
    if (static_cast<int>(threadIdx.x) < G::NCH) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < G::WAVES; ++w) s += wsum[w][threadIdx.x];
        enc_put(enc_place<G::NCH>(sums, grid, G::COLS, blockIdx.x), threadIdx.x, s);
        if constexpr (S::kInPlace) {  // (a quadratic chain)
            if (blockIdx.x == 0) enc_put(enc_place<G::NCH>(sums, grid, 0, sums.nb), threadIdx.x, chain[DIM + threadIdx.x]);
        }
    }
}

// Exclusive scan of the block sums in place: one workgroup, kScanThreads
// blocks of the chain (`cols` columns each) at a time.
constexpr int kScanThreads = 1024;

template <int NCH, typename S>
__global__ __launch_bounds__(kScanThreads) void k_enc_offsets(int64_t nb, int cols, float *__restrict__ grid, S sums) {
    constexpr int WAVES = kScanThreads / 64;
    __shared__ double wsum[WAVES][NCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double carry[NCH] = {};
    for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
        const int64_t b = b0 + threadIdx.x;
        float *__restrict__ p = enc_place<NCH>(sums, grid, cols, b);
        double v[NCH], incl[NCH];
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) incl[ch] = v[ch] = b < nb ? enc_get(p, ch) : 0.0;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double u = __shfl_up(incl[ch], off, 64);
                if (lane >= off) incl[ch] += u;
            }
            if (lane == 63) wsum[wave][ch] = incl[ch];
        }
        __syncthreads();
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            double pre = carry[ch];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {  // (unrolled: the LDS reads overlap)
                const double t = wsum[w][ch];
                carry[ch] += t;
                pre += w < wave ? t : 0.0;
            }
            if (b < nb) enc_put(p, ch, pre + (incl[ch] - v[ch]));
        }
        __syncthreads();
    }
}

// Writes the columns of a block: the endpoint in row k mod 2, the free texel
// in the other row.  Output [N+1][layers][2][DIM] (layers = ROWS - 1).
// DIRECT: the block adds up the chain before it itself (chains of a few
// blocks, in one launch); otherwise the sum before the block waits for it.
// (In place a block stages its columns before it writes the same, and reads no
// others.)
template <int DIM, int ROWS, int NT, bool DIRECT, typename S>
__global__ __launch_bounds__(NT) void k_enc_write(typename S::In chain, int64_t n_seg, typename S::Out grid, S sums) {
    using G = EncGeom<DIM, ROWS, NT>;
    constexpr int NCH = G::NCH;
    __shared__ float lds[G::LDS];
    __shared__ double wsum[G::WAVES][NCH], wpre[G::WAVES][NCH];
    const int64_t col0 = static_cast<int64_t>(blockIdx.x) * G::COLS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    enc_stage<DIM, ROWS, NT>(chain, n_seg, col0, lds);
    double pre[NCH] = {};
    if constexpr (!DIRECT) {
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) pre[ch] = enc_get(enc_place<NCH>(sums, grid, G::COLS, blockIdx.x), ch);
    } else {
        const int n = static_cast<int>(col0);  // a multiple of NT: column parity is the thread's
#pragma unroll 4
        for (int k = threadIdx.x; k < n; k += NT) {
            const float *__restrict__ p = chain + static_cast<int64_t>(k) * ROWS * DIM;
            auto row = [&](int j) { return p[j]; };
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) pre[ch] += enc_twice_mid<DIM, ROWS>(row, ch);
        }
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) pre[ch] = (threadIdx.x & 1) ? pre[ch] : -pre[ch];
    }
    __syncthreads();
    double ev[kEncPerThread][NCH], incl[NCH], own[NCH];
    enc_elems<DIM, ROWS, NT>(lds, n_seg, col0, ev);
    float A[kEncPerThread][DIM];
#pragma unroll
    for (int i = 0; i < kEncPerThread; ++i)
#pragma unroll
        for (int c = 0; c < DIM; ++c) A[i][c] = lds[threadIdx.x * (G::RUN | 1) + i * ROWS * DIM + c];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        own[ch] = ((ev[0][ch] + ev[1][ch]) + ev[2][ch]) + ev[3][ch];
        double v = own[ch];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double u = __shfl_up(v, off, 64);
            if (lane >= off) v += u;
        }
        incl[ch] = v;
        if (lane == 63) wsum[wave][ch] = v;
        if constexpr (DIRECT) {
            const double p = wave_sum64(pre[ch]);
            if (lane == 0) wpre[wave][ch] = p;
        }
    }
    __syncthreads();  // every thread has read its columns: their places may be overwritten
    float *run = lds + threadIdx.x * (G::OUT | 1);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        double y;  // M_0
        if constexpr (S::kInPlace) {
            y = enc_get(enc_place<NCH>(sums, grid, 0, sums.nb), ch);
        } else {
            typename S::In c0 = chain;
            auto row = [&](int j) { return c0[j]; };
            y = 0.5 * enc_twice_mid<DIM, ROWS>(row, ch);
        }
        if constexpr (!DIRECT) {
            y += pre[ch];
        } else {
#pragma unroll
            for (int w = 0; w < G::WAVES; ++w) y += wpre[w][ch];
        }
#pragma unroll
        for (int w = 0; w < G::WAVES; ++w)
            if (w < wave) y += wsum[w][ch];
        y += incl[ch] - own[ch];
        const int layer = ch / DIM, c = ch - layer * DIM;
#pragma unroll
        for (int i = 0; i < kEncPerThread; ++i) {
            float *col = run + (i * (ROWS - 1) + layer) * 2 * DIM;
            col[(i & 1) * DIM + c] = A[i][c];
            col[(1 - (i & 1)) * DIM + c] = static_cast<float>((i & 1) ? -y : y);
            y += ev[i][ch];
        }
    }
    __syncthreads();
    constexpr int GW = 2 * NCH;  // floats per grid column
    const int nf = static_cast<int>(min(static_cast<int64_t>(G::COLS), n_seg + 1 - col0)) * GW;
    float *__restrict__ dst = grid + col0 * GW;
#pragma unroll
    for (int i = 0; i < G::OUT / 4; ++i) {
        const int f = 4 * (threadIdx.x + i * NT), at = enc_at<G::OUT>(f);
        if (f + 4 <= nf) {
            enc_f4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = lds[at + e];
            *reinterpret_cast<enc_f4 *>(dst + f) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (f + e < nf) dst[f + e] = lds[at + e];
        }
    }
}

// Chains of up to kEncDirectCols columns go in one launch.  Chains of up to
// kEncSmallCols columns take blocks of 512 columns (128 threads), so that a
// chain of some ten thousand segments still spreads over the chip, longer ones
// blocks of 2048 (512 threads), whose sums are fewer to scan.
// (A cubic's columns are twice as wide: blocks of 1024.)
constexpr int kEncShortThreads = 128;
template <int ROWS>
constexpr int kEncLongThreads = ROWS == 2 ? 512 : 256;
constexpr int64_t kEncSmallCols = int64_t(1) << 18, kEncDirectCols = int64_t(1) << 15;

template <int DIM, int ROWS, int NT, typename S>
void launch_encode_blocks(const float *chain, int64_t n_seg, float *grid, S sums, hipStream_t s) {
    constexpr int COLS = EncGeom<DIM, ROWS, NT>::COLS, NCH = EncGeom<DIM, ROWS, NT>::NCH;
    const int64_t nb = (n_seg + COLS) / COLS;
    const dim3 blocks(static_cast<uint32_t>(nb));
    hipLaunchKernelGGL((k_enc_partials<DIM, ROWS, NT, S>), blocks, dim3(NT), 0, s, chain, n_seg, grid, sums);
    hipLaunchKernelGGL((k_enc_offsets<NCH, S>), dim3(1), dim3(kScanThreads), 0, s, nb, COLS, grid, sums);
    hipLaunchKernelGGL((k_enc_write<DIM, ROWS, NT, false, S>), blocks, dim3(NT), 0, s, chain, n_seg, grid, sums);
}

template <int DIM, int ROWS>
void launch_encode(const float *chain, int64_t n_seg, float *grid, EncInGrid sums, hipStream_t s) {
    constexpr int NL = kEncLongThreads<ROWS>, COLS = EncGeom<DIM, ROWS, NL>::COLS;
    if (n_seg + 1 <= kEncDirectCols)
        hipLaunchKernelGGL((k_enc_write<DIM, ROWS, NL, true, EncInGrid>), dim3(static_cast<uint32_t>((n_seg + COLS) / COLS)),
                           dim3(NL), 0, s, chain, n_seg, grid, sums);
    else if (n_seg + 1 <= kEncSmallCols)
        launch_encode_blocks<DIM, ROWS, kEncShortThreads>(chain, n_seg, grid, sums, s);
    else
        launch_encode_blocks<DIM, ROWS, NL>(chain, n_seg, grid, sums, s);
}

// In place: long blocks whatever the size, as the workspace is counted in them.
template <int DIM, int ROWS>
void launch_encode(const float *chain, int64_t n_seg, float *grid, EncInPlace sums, hipStream_t s) {
    launch_encode_blocks<DIM, ROWS, kEncLongThreads<ROWS>>(chain, n_seg, grid, sums, s);
}

template <int ROWS, typename S>
void launch_encode_dim(int dim, const float *chain, int64_t n_seg, float *grid, S sums, hipStream_t s) {
    switch (dim) {
        case 1: launch_encode<1, ROWS>(chain, n_seg, grid, sums, s); break;
        case 2: launch_encode<2, ROWS>(chain, n_seg, grid, sums, s); break;
        case 3: launch_encode<3, ROWS>(chain, n_seg, grid, sums, s); break;
        default: launch_encode<4, ROWS>(chain, n_seg, grid, sums, s); break;
    }
}

// Longest chain bz_encode_piecewise_noalloc takes, part of its interface: its
// blocks' sums fit g_enc_scratch.
constexpr int64_t kEncLongCols = EncGeom<1, 2, kEncLongThreads<2>>::COLS;
int64_t noalloc_max_seg(int dim) { return kEncScratchDoubles / dim * kEncLongCols - 1; }

}  // namespace
}  // namespace bzi

using namespace bzi;

extern "C" {

// alloc: whether a chain encoded in place may take a workspace from the stream's
// memory; else it takes the library's.
static int encode_chain(const char *fn, const float *chain, int64_t n_seg, int dim, int cubic, bool alloc, float *grid,
                        bz_stream stream) {
    if (dim < 1 || dim > kMaxDim) return fail(BZ_ERR_SHAPE, "%s: dim %d", fn, dim);
    if (n_seg < 0 || n_seg > (int64_t(1) << 40)) return fail(BZ_ERR_SHAPE, "%s: n_seg %lld", fn, (long long)n_seg);
    if (n_seg == 0) return BZ_OK;
    if (!chain || !grid) return fail(BZ_ERR_NULL, "%s: chain and grid are required", fn);
    if (!aligned(chain, 4) || !aligned(grid, 4)) return fail(BZ_ERR_ALIGN, "%s: misaligned", fn);
    const hipStream_t s = as_stream(stream);
    if (cubic) {
        launch_encode_dim<3>(dim, chain, n_seg, grid, EncInGrid{}, s);
    } else if (grid != chain) {
        launch_encode_dim<2>(dim, chain, n_seg, grid, EncInGrid{}, s);
    } else {
        EncInPlace at{nullptr, (n_seg + kEncLongCols) / kEncLongCols};
        if (alloc) {
            const hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&at.ws), sizeof(double) * (at.nb + 1) * dim, s);
            if (e == hipErrorOutOfMemory) return fail(BZ_ERR_NOMEM, "%s: workspace", fn);
            BZ_CHECK_HIP(e);
        }
        launch_encode_dim<2>(dim, chain, n_seg, grid, at, s);
        const hipError_t le = hipGetLastError();
        if (alloc) BZ_CHECK_HIP(hipFreeAsync(at.ws, s));
        if (le != hipSuccess) return hip_fail(le, fn);
    }
    BZ_CHECK_LAUNCH(fn);
    return BZ_OK;
}

int bz_encode_piecewise_noalloc(const float *chain, int64_t n_seg, int dim, float *grid, bz_stream stream) {
    return guarded("bz_encode_piecewise_noalloc", [&]() -> int {
        const char *fn = "bz_encode_piecewise_noalloc";
        if (dim < 1 || dim > kMaxDim) return fail(BZ_ERR_SHAPE, "%s: dim %d", fn, dim);
        if (n_seg < 0 || n_seg > noalloc_max_seg(dim))
            return fail(BZ_ERR_SHAPE, "%s: n_seg %lld outside 0..%lld, the workspace limit for dim %d", fn,
                        (long long)n_seg, (long long)noalloc_max_seg(dim), dim);
        return encode_chain(fn, chain, n_seg, dim, 0, false, grid, stream);
    });
}

int bz_encode_piecewise(const float *chain, int64_t n_seg, int dim, float *grid, bz_stream stream) {
    return guarded("bz_encode_piecewise",
                   [&]() -> int { return encode_chain("bz_encode_piecewise", chain, n_seg, dim, 0, true, grid, stream); });
}

int bz_encode_piecewise_cubic(const float *chain, int64_t n_seg, int dim, float *grid, bz_stream stream) {
    return guarded("bz_encode_piecewise_cubic", [&]() -> int {
        return encode_chain("bz_encode_piecewise_cubic", chain, n_seg, dim, 1, true, grid, stream);
    });
}

}  // extern "C"
