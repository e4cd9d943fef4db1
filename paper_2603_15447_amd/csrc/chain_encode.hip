// Zig-zag encoder of C0 piecewise chains (Sec. 2.1, Eq. 2, Fig. 2): the free
// texels of a chain of N segments are fixed by x_0 = M_0 and x_k + x_{k+1} =
// 2 M_k, an alternating prefix sum over the middle points, evaluated here as
// an FP64 block scan (per-block partials, then one pass that adds up the
// partials before its block, scans its own columns and writes them): every
// texel is one FP32 rounding of an FP64 prefix sum, where an FP32 recurrence
// x_{k+1} = 2 M_k - x_k would let the rounding error grow with k.
#include <mutex>

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
// different banks.  (Threads reading their columns from global memory and
// writing them there, a column pitch of 2*DIM floats apart, took 85 us for the
// last pass alone at 2^20 3D segments, whose 50 MB a copy moves in 10.)
constexpr int kEncPerThread = 4;

template <int DIM, int ROWS, int NT>
struct EncGeom {
    static constexpr int NCH = DIM * (ROWS - 1);
    static constexpr int COLS = NT * kEncPerThread;         // columns per block
    static constexpr int RUN = kEncPerThread * ROWS * DIM;  // floats of a thread's columns
    static constexpr int PITCH = RUN | 1;
    static constexpr int N = COLS * ROWS * DIM + (ROWS == 3 ? DIM : 0);  // floats staged
    static constexpr int LDS = NT * PITCH + (ROWS == 3 ? DIM : 0);
    static constexpr int WAVES = NT / 64;
    // LDS word of float f of the block's rows
    static __device__ __forceinline__ int at(int f) { return f + (PITCH - RUN) * (f / RUN); }
};

typedef float enc_f4 __attribute__((ext_vector_type(4), aligned(4)));

// Rows of the block's columns [col0, col0 + COLS), zero past the chain's end.
template <int DIM, int ROWS, int NT>
__device__ __forceinline__ void enc_stage(const float *__restrict__ chain, int64_t n_seg, int64_t col0, float *lds) {
    using G = EncGeom<DIM, ROWS, NT>;
    const int64_t first = col0 * ROWS * DIM, total = (n_seg * ROWS + 1) * DIM;
    const float *__restrict__ src = chain + first;
    const int avail = static_cast<int>(min(static_cast<int64_t>(G::N), total - first));
    for (int f = 4 * threadIdx.x; f < G::N; f += 4 * NT) {
        float v[4] = {};
        if (f + 4 <= avail) {
            const enc_f4 x = *reinterpret_cast<const enc_f4 *>(src + f);
            v[0] = x[0], v[1] = x[1], v[2] = x[2], v[3] = x[3];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (f + e < avail) v[e] = src[f + e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (G::N % 4 == 0 || f + e < G::N) lds[G::at(f + e)] = v[e];
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
        const int f0 = (threadIdx.x * kEncPerThread + i) * ROWS * DIM;
        auto row = [&](int j) { return lds[G::at(f0 + j)]; };
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

template <int DIM, int ROWS, int NT>
__global__ __launch_bounds__(NT) void k_enc_partials(const float *__restrict__ chain, int64_t n_seg,
                                                     double *__restrict__ partial) {
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
        partial[static_cast<int64_t>(blockIdx.x) * G::NCH + threadIdx.x] = s;
    }
}

// Exclusive scan of the block partials in place (one block, serial over
// chunks), for chains of so many blocks that each block adding up its
// predecessors' partials would read more than the chain itself.
__global__ __launch_bounds__(kBlock) void k_enc_offsets(int nch, int64_t nb, double *__restrict__ partial) {
    __shared__ double wsum[kBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int ch = 0; ch < nch; ++ch) {
        double carry = 0.0;
        for (int64_t b0 = 0; b0 < nb; b0 += kBlock) {
            const int64_t b = b0 + threadIdx.x;
            const double v = b < nb ? partial[b * nch + ch] : 0.0;
            double incl = v;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double u = __shfl_up(incl, off, 64);
                if (lane >= off) incl += u;
            }
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            double pre = carry;
            for (int w = 0; w < wave; ++w) pre += wsum[w];
            if (b < nb) partial[b * nch + ch] = pre + (incl - v);
            for (int w = 0; w < kBlock / 64; ++w) carry += wsum[w];
            __syncthreads();
        }
    }
}

// Where a block finds the sum of the elements before its columns.
enum {
    kEncDirect = 0,   // adds up the chain before it (no workspace: chains of a few blocks)
    kEncSelfSum = 1,  // adds up the partials before it
    kEncScanned = 2   // k_enc_offsets has scanned the partials
};

// Writes the columns of a block: the endpoint in row k mod 2, the free texel
// in the other row.  Output [N+1][layers][2][DIM] (layers = ROWS - 1).
template <int DIM, int ROWS, int NT, int MODE>
__global__ __launch_bounds__(NT) void k_enc_write(const float *__restrict__ chain, int64_t n_seg,
                                                  const double *__restrict__ partial, float *__restrict__ grid) {
    using G = EncGeom<DIM, ROWS, NT>;
    constexpr int NCH = G::NCH;
    __shared__ float lds[G::LDS];
    __shared__ double wsum[G::WAVES][NCH], wpre[G::WAVES][NCH];
    const int64_t col0 = static_cast<int64_t>(blockIdx.x) * G::COLS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    enc_stage<DIM, ROWS, NT>(chain, n_seg, col0, lds);
    double pre[NCH] = {};
    if constexpr (MODE == kEncSelfSum) {
        const int nb = static_cast<int>(blockIdx.x);
#pragma unroll 2
        for (int b = threadIdx.x; b < nb; b += NT)
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) pre[ch] += partial[static_cast<int64_t>(b) * NCH + ch];
    } else if constexpr (MODE == kEncDirect) {
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
        if constexpr (MODE != kEncScanned) {
            const double p = wave_sum64(pre[ch]);
            if (lane == 0) wpre[wave][ch] = p;
        }
    }
    __syncthreads();  // every thread has read its elements: their places may be overwritten
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const float *__restrict__ c0 = chain;
        auto row = [&](int j) { return c0[j]; };
        double y = 0.5 * enc_twice_mid<DIM, ROWS>(row, ch);  // M_0
        if constexpr (MODE == kEncScanned) {
            y += partial[static_cast<int64_t>(blockIdx.x) * NCH + ch];
        } else {
#pragma unroll
            for (int w = 0; w < G::WAVES; ++w) y += wpre[w][ch];
        }
#pragma unroll
        for (int w = 0; w < G::WAVES; ++w)
            if (w < wave) y += wsum[w][ch];
        y += incl[ch] - own[ch];
#pragma unroll
        for (int i = 0; i < kEncPerThread; ++i) {
            const int f0 = (threadIdx.x * kEncPerThread + i) * ROWS * DIM;
            lds[G::at(f0 + DIM + ch)] = static_cast<float>((i & 1) ? -y : y);  // rows 1.. of the column: channel order
            y += ev[i][ch];
        }
    }
    __syncthreads();
    // grid float f of the block: column, layer, row, coordinate
    constexpr int GW = 2 * NCH;  // floats per grid column
    const int64_t cols = min(static_cast<int64_t>(G::COLS), n_seg + 1 - col0);
    const int nf = static_cast<int>(cols) * GW;
    float *__restrict__ dst = grid + col0 * GW;
    auto texel = [&](int f) {
        const int k = f / GW, r = f - k * GW;
        const int layer = r / (2 * DIM), q = r - layer * 2 * DIM;
        const int rw = q >= DIM, c = q - rw * DIM;
        return lds[G::at(k * ROWS * DIM + (rw == (k & 1) ? c : DIM + layer * DIM + c))];
    };
    for (int f = 4 * threadIdx.x; f < nf; f += 4 * NT) {
        enc_f4 v;
        if (GW % 4 == 0 || f + 4 <= nf) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = texel(f + e);
            *reinterpret_cast<enc_f4 *>(dst + f) = v;
        } else {
            for (int e = 0; f + e < nf; ++e) dst[f + e] = texel(f + e);
        }
    }
}

// Partials of chains of up to kEncSmallCols columns come from blocks of 512
// columns (128 threads), so that a chain of a few thousand segments still
// spreads over the chip; longer chains take blocks of 2048 (512 threads), and
// from kEncSelfSumMax blocks on one more launch scans the partials.  Chains of
// up to kEncDirectCols columns go in one launch without a workspace.
constexpr int kEncLongThreads = 512, kEncShortThreads = 128;
constexpr int kEncPerBlock = kEncLongThreads * kEncPerThread;  // columns of a long chain's block
constexpr int64_t kEncSmallCols = int64_t(1) << 18, kEncDirectCols = 4 * kEncPerBlock, kEncSelfSumMax = 4096;

struct EncPlan {
    int64_t cols;  // columns per block
    int64_t nb;    // blocks
    int mode;
};

EncPlan enc_plan(int64_t n_seg) {
    const int64_t n = n_seg + 1;
    const bool direct = n <= kEncDirectCols;
    const int64_t cols = !direct && n <= kEncSmallCols ? kEncShortThreads * kEncPerThread : kEncPerBlock;
    const int64_t nb = (n + cols - 1) / cols;
    return {cols, nb, direct ? kEncDirect : nb <= kEncSelfSumMax ? kEncSelfSum : kEncScanned};
}

template <int DIM, int ROWS>
void launch_encode(const EncPlan &p, const float *chain, int64_t n_seg, double *partial, float *grid, hipStream_t s) {
    constexpr int NL = kEncLongThreads, NS = kEncShortThreads;
    const dim3 blocks(static_cast<uint32_t>(p.nb));
    if (p.mode == kEncDirect) {
        hipLaunchKernelGGL((k_enc_write<DIM, ROWS, NL, kEncDirect>), blocks, dim3(NL), 0, s, chain, n_seg, partial, grid);
    } else if (p.cols != kEncPerBlock) {
        hipLaunchKernelGGL((k_enc_partials<DIM, ROWS, NS>), blocks, dim3(NS), 0, s, chain, n_seg, partial);
        hipLaunchKernelGGL((k_enc_write<DIM, ROWS, NS, kEncSelfSum>), blocks, dim3(NS), 0, s, chain, n_seg, partial, grid);
    } else {
        hipLaunchKernelGGL((k_enc_partials<DIM, ROWS, NL>), blocks, dim3(NL), 0, s, chain, n_seg, partial);
        if (p.mode == kEncSelfSum) {
            hipLaunchKernelGGL((k_enc_write<DIM, ROWS, NL, kEncSelfSum>), blocks, dim3(NL), 0, s, chain, n_seg, partial, grid);
        } else {
            hipLaunchKernelGGL(k_enc_offsets, dim3(1), dim3(kBlock), 0, s, DIM * (ROWS - 1), p.nb, partial);
            hipLaunchKernelGGL((k_enc_write<DIM, ROWS, NL, kEncScanned>), blocks, dim3(NL), 0, s, chain, n_seg, partial, grid);
        }
    }
}

template <int ROWS>
void launch_encode_dim(int dim, const EncPlan &p, const float *chain, int64_t n_seg, double *partial, float *grid,
                       hipStream_t s) {
    switch (dim) {
        case 1: launch_encode<1, ROWS>(p, chain, n_seg, partial, grid, s); break;
        case 2: launch_encode<2, ROWS>(p, chain, n_seg, partial, grid, s); break;
        case 3: launch_encode<3, ROWS>(p, chain, n_seg, partial, grid, s); break;
        default: launch_encode<4, ROWS>(p, chain, n_seg, partial, grid, s); break;
    }
}

}  // namespace

// Workspace of the allocation-free encoder: the block partials (one double
// per block of kEncPerBlock columns and channel) in a file-scope device array.
// Each device holds its own copy until the process ends; host code reaches it
// only through the device address looked up per device below (the array's
// name in host code is a host-side stand-in, not a device address).
constexpr int64_t kEncScratchDoubles = int64_t(1) << 18;  // 2 MiB
static __device__ __align__(256) double scratch[kEncScratchDoubles];

namespace {

// Largest chain the workspace holds: nb * dim <= kEncScratchDoubles with
// nb = ceil((n_seg + 1) / kEncPerBlock).  (Chains of up to kEncSmallCols
// columns take smaller blocks, at most 512 of them.)
int64_t noalloc_max_seg(int dim) { return (kEncScratchDoubles / dim) * kEncPerBlock - 1; }

constexpr int kScratchMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kScratchMaxDevices] = {};

// Device address of the current device's scratch array, looked up once per
// device (with that device current) and kept.
int scratch_address(const char *fn, double **out) {
    int dev = 0;
    BZ_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kScratchMaxDevices) return fail(BZ_ERR_UNSUPPORTED, "%s: device %d", fn, dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return BZ_OK;
}

}  // namespace
}  // namespace bzi

using namespace bzi;

extern "C" {

// ws: caller-provided workspace of at least nb*nch doubles, or NULL for a
// stream-ordered allocation freed after the launches (none is made for chains
// that go in one launch).
static int encode_chain(const char *fn, const float *chain, int64_t n_seg, int dim, int cubic, float *grid,
                        bz_stream stream, double *ws = nullptr) {
    if (dim < 1 || dim > kMaxDim) return fail(BZ_ERR_SHAPE, "%s: dim %d", fn, dim);
    if (n_seg < 0 || n_seg > (int64_t(1) << 40)) return fail(BZ_ERR_SHAPE, "%s: n_seg %lld", fn, (long long)n_seg);
    if (n_seg == 0) return BZ_OK;
    if (!chain || !grid) return fail(BZ_ERR_NULL, "%s: chain and grid are required", fn);
    if (!aligned(chain, 4) || !aligned(grid, 4)) return fail(BZ_ERR_ALIGN, "%s: misaligned", fn);
    const hipStream_t s = as_stream(stream);
    const int nch = dim * (cubic ? 2 : 1);
    const EncPlan plan = enc_plan(n_seg);
    double *partial = ws;
    const bool own = !ws && plan.mode != kEncDirect;
    if (own) {
        hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&partial), sizeof(double) * plan.nb * nch, s);
        if (e == hipErrorOutOfMemory) return fail(BZ_ERR_NOMEM, "%s: workspace", fn);
        BZ_CHECK_HIP(e);
    }
    // every partial is written by k_enc_partials before it is read: the
    // workspace needs no clearing
    if (cubic) launch_encode_dim<3>(dim, plan, chain, n_seg, partial, grid, s);
    else launch_encode_dim<2>(dim, plan, chain, n_seg, partial, grid, s);
    const hipError_t le = hipGetLastError();
    if (own) BZ_CHECK_HIP(hipFreeAsync(partial, s));
    if (le != hipSuccess) return hip_fail(le, fn);
    return BZ_OK;
}

int bz_encode_piecewise_noalloc(const float *chain, int64_t n_seg, int dim, float *grid, bz_stream stream) {
    return guarded("bz_encode_piecewise_noalloc", [&]() -> int {
        const char *fn = "bz_encode_piecewise_noalloc";
        if (dim < 1 || dim > kMaxDim) return fail(BZ_ERR_SHAPE, "%s: dim %d", fn, dim);
        if (n_seg < 0 || n_seg > noalloc_max_seg(dim))
            return fail(BZ_ERR_SHAPE, "%s: n_seg %lld outside 0..%lld, the workspace limit for dim %d", fn,
                        (long long)n_seg, (long long)noalloc_max_seg(dim), dim);
        if (n_seg == 0) return BZ_OK;
        double *ws = nullptr;
        const int rc = scratch_address(fn, &ws);
        if (rc) return rc;
        return encode_chain(fn, chain, n_seg, dim, 0, grid, stream, ws);
    });
}


int bz_encode_piecewise(const float *chain, int64_t n_seg, int dim, float *grid, bz_stream stream) {
    return guarded("bz_encode_piecewise",
                   [&]() -> int { return encode_chain("bz_encode_piecewise", chain, n_seg, dim, 0, grid, stream); });
}

int bz_encode_piecewise_cubic(const float *chain, int64_t n_seg, int dim, float *grid, bz_stream stream) {
    return guarded("bz_encode_piecewise_cubic", [&]() -> int {
        return encode_chain("bz_encode_piecewise_cubic", chain, n_seg, dim, 1, grid, stream);
    });
}

}  // extern "C"
