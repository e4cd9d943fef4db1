// Separable tensor-product kernels shared by the Bernstein (tensor.hip) and
// per-axis Seiler (tensor_seiler.hip) evaluators of surfaces and volumes
// (Sec. 2.2: the order splits over the parameter axes).  The contraction is
// the same for both; only the per-axis basis differs.
//
//  k_tensor_grid   nu x nv uniform grids: a workgroup contracts the net with
//                  the v basis once per grid column (isoline coefficients
//                  R_i(v_b), shared through LDS with the u basis of its rows),
//                  then du+1 FMAs per coordinate and point.
//  k_tensor_points one object per wavefront, random (u,v[,w]) per query,
//                  4 queries per lane, separable contraction w -> v -> u.
#pragma once
#include "curves_impl.h"

namespace bzi {
namespace {

// Per-axis basis: Bernstein for control points, or the Seiler basis for
// per-axis Seiler terms stored [b0, bd, d1, d_{d-1}, d2, ...] (Sec. 3): the
// Seiler recursion L(b0,bd,t) + st (L(d1,d_{d-1},t) + st (...)) is linear in
// the terms with coefficients 1-t, t, st(1-t), st t, (st)^2(1-t), ...,
// and (st)^(d/2) for the middle term of even degree.
enum { kBasisBernstein = 0, kBasisSeiler = 1 };

template <int D>
__device__ __forceinline__ void seiler_basis(float t, float (&B)[D + 1]) {
    const float s = 1.0f - t, st = s * t;
    B[0] = s;
    if constexpr (D >= 1) B[1] = t;
    float p = 1.0f;
#pragma unroll
    for (int i = 1; 2 * i + 1 <= D; ++i) {
        p *= st;
        B[2 * i] = p * s;
        B[2 * i + 1] = p * t;
    }
    if constexpr (D >= 2 && D % 2 == 0) {
        float m = 1.0f;
#pragma unroll
        for (int i = 0; i < D / 2; ++i) m *= st;
        B[D] = m;
    }
}

template <int D, int BASIS>
__device__ __forceinline__ void basis_at(float x, float (&B)[D + 1]) {
    if constexpr (BASIS == kBasisSeiler) seiler_basis<D>(x, B);
    else bernstein_basis<D>(x, B);
}

// ------------------------------------------------------------------ VALU grid
// Uniform nu x nv grids.  A workgroup takes `chunk` consecutive points of the
// output: of the whole sequence of patches when a patch's rows and columns
// both fit one workgroup's tables (the chunk may then cover several patches,
// or parts of them), else of one strip of `cb` columns of one patch.  The u
// basis of its rows and the isoline coefficients R[c][i] = sum_j Bv_j(b)
// P[c][i][j] of its columns are formed once and shared through LDS; a point is
// then one row of the u basis, one column of R and du+1 FMAs per coordinate.
// The output's writes bound it: the LDS reads (16 bytes of the u basis and 16
// per coordinate of R, each padded to whole 16-byte vectors) and about 35
// vector instructions per 64 points both allow twice the write rate.
struct GridArgs {
    int nu, nv;
    int cb, strips;         // columns of a strip, strips per patch
    int chunk;              // points per workgroup
    int rows, slots;        // table capacities: rows of the u basis, patches per chunk
    uint32_t per_strip;     // workgroups per strip; 0: chunks of the whole sequence
    uint32_t n;             // points of the sequence, or of one strip
    uint32_t npts;          // points of a patch, or of one strip
    FastDiv div_cb, div_npts;
    int64_t plane, o0;
    int same;               // whole sequence: the planes lie alike to the 64-byte lines
};

// Floats of one (coordinate, column) or row entry of the LDS tables.
template <int DU>
constexpr int kGridPad = (DU + 4) / 4 * 4;

// The control net of patch k of the workgroup, widened.
template <int N, typename T>
__device__ __forceinline__ void load_net(const T *__restrict__ p, float (&v)[N]) {
    if constexpr (std::is_same<T, float>::value) {
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int e = 0; e + 4 <= N; e += 4) {
            const f4u x = *reinterpret_cast<const f4u *>(p + e);
            v[e] = x[0], v[e + 1] = x[1], v[e + 2] = x[2], v[e + 3] = x[3];
        }
#pragma unroll
        for (int e = N / 4 * 4; e < N; ++e) v[e] = p[e];
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = to_f32<T>(p[e]);
    }
}

template <int DU, int DV, int DIM, typename T, int BASIS>
__global__ __launch_bounds__(kBlock) void k_tensor_grid(const T *__restrict__ ctrl, GridArgs g, float *__restrict__ out) {
    constexpr int NCP = (DU + 1) * (DV + 1), PAD = kGridPad<DU>;
    extern __shared__ __align__(16) float lds[];
    float *__restrict__ tab_u = lds;                   // [rows][PAD]
    float *__restrict__ tab_r = lds + PAD * g.rows;    // [DIM][slots*cb][PAD]
    // [q0, q0 + n): the chunk in the sequence (or strip); o: its first patch,
    // s0: its first point there
    const int64_t patch_pts = static_cast<int64_t>(g.nu) * g.nv;
    float *__restrict__ seq = out + g.o0 * patch_pts;
    uint32_t o, q0, s0, sh = 0;
    int b0 = 0;
    if (g.per_strip == 0) {
        // every chunk but the first begins on a 128-byte line of plane 0, or of
        // each plane (then up to 31 points earlier, which the tables cover)
        sh = g.same ? line_offset(seq) : 31;
        const uint32_t at = blockIdx.x * g.chunk;
        q0 = at > sh ? at - sh : 0;
        o = fdiv(q0, g.div_npts);
        s0 = q0 - o * g.npts;
    } else {
        const uint32_t r = blockIdx.x / g.per_strip;
        o = r / g.strips;
        b0 = static_cast<int>(r - o * g.strips) * g.cb;
        s0 = q0 = (blockIdx.x - r * g.per_strip) * g.chunk;
    }
    const uint32_t end = min(g.n, g.per_strip == 0 ? (blockIdx.x + 1) * g.chunk - (g.same ? sh : 0) : q0 + g.chunk);
    const int n = static_cast<int>(end - q0);
    if (n <= 0) return;
    const int n_slots = static_cast<int>(fdiv(s0 + n - 1, g.div_npts)) + 1;
    const int cols = min(g.cb, g.nv - b0);
    // rows of the chunk: those of its one patch that it touches, or all
    const int a_lo = n_slots == 1 ? static_cast<int>(fdiv(s0, g.div_cb)) : 0;
    const int a_hi = n_slots == 1 ? static_cast<int>(fdiv(s0 + n - 1, g.div_cb)) : g.nu - 1;
    const float du_den = g.nu > 1 ? static_cast<float>(g.nu - 1) : 1.0f;
    const float dv_den = g.nv > 1 ? static_cast<float>(g.nv - 1) : 1.0f;
    const T *__restrict__ P = ctrl + static_cast<size_t>(o) * DIM * NCP;
    const int n_cols = g.slots * g.cb;
    // (one patch: its net is the same for all threads and comes in by scalar loads)
    auto contract = [&](const T *__restrict__ net, int e, int b) {
        float N[DIM * NCP], Bv[DV + 1];
        load_net<DIM * NCP>(net, N);
        basis_at<DV, BASIS>(static_cast<float>(b0 + b) / dv_den, Bv);
#pragma unroll
        for (int c = 0; c < DIM; ++c)
#pragma unroll
            for (int i = 0; i <= DU; ++i) {
                float acc = Bv[0] * N[c * NCP + i * (DV + 1)];
#pragma unroll
                for (int j = 1; j <= DV; ++j) acc = __builtin_fmaf(Bv[j], N[c * NCP + i * (DV + 1) + j], acc);
                tab_r[(c * n_cols + e) * PAD + i] = acc;
            }
    };
    if (n_slots == 1) {
        if (static_cast<int>(threadIdx.x) < g.cb) contract(P, threadIdx.x, threadIdx.x);
    } else {
        for (int e = threadIdx.x; e < n_slots * g.cb; e += kBlock) {
            const int k = static_cast<int>(fdiv(e, g.div_cb));
            contract(P + static_cast<size_t>(k) * DIM * NCP, e, e - k * g.cb);
        }
    }
    // the u basis from the block's other end: its last waves have no columns while there are few
    for (int a = kBlock - 1 - threadIdx.x; a <= a_hi - a_lo; a += kBlock) {
        float Bu[DU + 1];
        basis_at<DU, BASIS>(static_cast<float>(a_lo + a) / du_den, Bu);
#pragma unroll
        for (int i = 0; i <= DU; ++i) tab_u[a * PAD + i] = Bu[i];
    }
    __syncthreads();
    // coordinate c of the point in row a, column b of patch k of the chunk
    auto point = [&](int c, const float (&Bu)[DU + 1], uint32_t k, uint32_t b) {
        float R[DU + 1];
#pragma unroll
        for (int i = 0; i <= DU; ++i) R[i] = tab_r[(c * n_cols + k * g.cb + b) * PAD + i];
        return dot_basis<DU>(Bu, R);
    };
    auto row = [&](uint32_t a, float (&Bu)[DU + 1]) {
#pragma unroll
        for (int i = 0; i <= DU; ++i) Bu[i] = tab_u[(a - a_lo) * PAD + i];
    };
    if (g.per_strip != 0) {
        float *__restrict__ ob = seq + o * patch_pts + b0;
        for (int p = threadIdx.x; p < n; p += kBlock) {
            const uint32_t a = fdiv(s0 + p, g.div_cb), b = s0 + p - a * g.cb;
            if (static_cast<int>(b) >= cols) continue;  // a patch's last strip is narrower
            float Bu[DU + 1];
            row(a, Bu);
#pragma unroll
            for (int c = 0; c < DIM; ++c) ob[c * g.plane + a * g.nv + b] = point(c, Bu, 0, b);
        }
        return;
    }
    // whole sequence: in plain order where the planes lie alike, else by way of
    // LDS, from where each plane's own points, up to 31 apart, are stored so that
    // every wave fills whole lines of it
    float *__restrict__ buf = tab_r + PAD * DIM * n_cols;  // [DIM][chunk + 32]
    const int pitch = g.chunk + 32;
    // every point of the chunk; a full chunk's four per thread without bounds
    // checks between them, so that their LDS reads overlap (the one point too
    // many of a relayed chunk is its last again)
    auto each = [&](auto f) {
        if (n >= 4 * kBlock - 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) f(min(static_cast<int>(threadIdx.x) + i * kBlock, n - 1));
        } else {
            for (int p = threadIdx.x; p < n; p += kBlock) f(p);
        }
    };
    auto points = [&](auto same) {
        auto put = [&](int c, int p, float v) {
            if constexpr (decltype(same)::value) st_stream(seq + c * g.plane + q0 + p, v);
            else buf[c * pitch + p] = v;
        };
        if (n_slots == 1 && kBlock % g.cb == 0) {
            // one patch and whole rows per step: a thread stays in its column and
            // keeps that column's coefficients (32 x 32 grids: 42 -> 35 us)
            const uint32_t a = fdiv(s0 + threadIdx.x, g.div_cb), b = s0 + threadIdx.x - a * g.cb;
            const uint32_t step = kBlock / g.cb;
            float R[DIM][DU + 1];
#pragma unroll
            for (int c = 0; c < DIM; ++c)
#pragma unroll
                for (int i = 0; i <= DU; ++i) R[c][i] = tab_r[(c * n_cols + b) * PAD + i];
            auto step_to = [&](int i) {
                float Bu[DU + 1];
                row(a + i * step, Bu);
#pragma unroll
                for (int c = 0; c < DIM; ++c) put(c, threadIdx.x + i * kBlock, dot_basis<DU>(Bu, R[c]));
            };
            if (n == 4 * kBlock) {
#pragma unroll
                for (int i = 0; i < 4; ++i) step_to(i);
            } else {
                for (int i = 0; static_cast<int>(threadIdx.x) + i * kBlock < n; ++i) step_to(i);
            }
            return;
        }
        each([&](int p) {
            const uint32_t k = fdiv(s0 + p, g.div_npts), r = s0 + p - k * g.npts;
            const uint32_t a = fdiv(r, g.div_cb), b = r - a * g.cb;
            float Bu[DU + 1];
            row(a, Bu);
#pragma unroll
            for (int c = 0; c < DIM; ++c) put(c, p, point(c, Bu, k, b));
        });
    };
    if (g.same) {
        points(std::true_type{});
        return;
    }
    points(std::false_type{});
    __syncthreads();
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        float *__restrict__ oc = seq + c * g.plane;
        const uint32_t first = blockIdx.x * g.chunk - line_offset(oc);  // may lie before 0: wraps
        for (uint32_t p = threadIdx.x; p < static_cast<uint32_t>(g.chunk); p += kBlock) {
            const uint32_t q = first + p;
            if (q < g.n) st_stream(oc + q, buf[c * pitch + (q - q0)]);
        }
    }
}

// Layout of a grid call.  1024 points per workgroup (four per thread): short
// workgroups write faster than long ones (32 x 32 grids of 16384 bicubic 3D
// patches: 34.7 us with 1024, 37 with 2048, 42 with 4096, 47 with 512), fewer
// points where a call is too small to give every CU four workgroups or the
// tables of so many points would leave a CU too few workgroups.
// Results go past the caches, for which each wave's store has to fill whole
// lines: chunks begin on a line, and where the planes don't lie alike (their
// distance is no multiple of 64 bytes), each plane's part of the chunk does.
// 16384 patches of 33 x 33 points: 75 us with a patch per workgroup from its
// first point on, 35 now; one patch more, whose planes don't lie alike: 48, and
// 53 with ordinary stores in the order of evaluation.
constexpr size_t kGridTableFloats = 10240;

template <int DU, int DIM>
size_t grid_floats(const GridArgs &g) {
    return kGridPad<DU> * (g.rows + static_cast<size_t>(DIM) * g.slots * g.cb) +
           (g.per_strip == 0 && !g.same ? static_cast<size_t>(DIM) * (g.chunk + 32) : 0);
}

template <int DU, int DIM>
GridArgs grid_args(int nu, int nv, int64_t n_obj, int64_t plane) {
    GridArgs g{};
    g.nu = nu;
    g.nv = nv;
    g.plane = plane;
    g.same = plane % 16 == 0 || DIM == 1;
    const int64_t npts = static_cast<int64_t>(nu) * nv, total = n_obj * npts;
    const int want = total >= int64_t(1024) * 256 ? 1024 : total >= int64_t(512) * 256 ? 512 : 256;
    bool seq = false;
    if (nu <= kBlock && nv <= kBlock) {
        g.strips = 1;
        g.cb = nv;
        g.npts = static_cast<uint32_t>(npts);
        g.rows = nu;
        for (int chunk = want; chunk >= 256 && !seq; chunk /= 2) {
            g.chunk = g.same ? chunk : chunk - 32;  // with the planes' own first points a whole number per thread
            g.slots = static_cast<int>((g.chunk + 31 + npts - 2) / npts + 1);
            seq = grid_floats<DU, DIM>(g) <= kGridTableFloats;
        }
    }
    if (!seq) {  // long rows or columns, or rows too few to share a column's contraction
        g.strips = (nv + kBlock - 1) / kBlock;
        g.cb = (nv + g.strips - 1) / g.strips;
        g.strips = (nv + g.cb - 1) / g.cb;
        g.chunk = std::max(want, 8 * g.cb);  // a strip's columns are contracted once per chunk
        g.npts = g.n = static_cast<uint32_t>(nu) * g.cb;
        g.per_strip = (g.n + g.chunk - 1) / g.chunk;
        g.slots = 1;
        g.rows = std::min(nu, g.chunk / g.cb + 2);
    }
    g.div_cb = make_fastdiv(g.cb);
    g.div_npts = make_fastdiv(g.npts);
    return g;
}

// ------------------------------------------------------------------ VALU points
// One wavefront per object, 4 queries per lane at a time: the object's
// control points are wave-uniform (scalar loads into SGPRs) and each one
// feeds the FMAs of 4 queries.  Separable contraction w -> v -> u.
constexpr int kPtsQ = 4;

template <int DU, int DV, int DW, int DIM, typename T, int BASIS>
__global__ __launch_bounds__(kBlock) void k_tensor_points(const T *__restrict__ ctrl, const float *__restrict__ uvw,
                                                          int64_t n_per, uint32_t n_obj, float *__restrict__ out,
                                                          int64_t plane, int64_t o0) {
    constexpr int NCP = (DU + 1) * (DV + 1) * (DW + 1);
    constexpr int NPAR = DW > 0 ? 3 : 2;
    const uint32_t o = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6));
    if (o >= n_obj) return;
    const int lane = threadIdx.x & 63;
    const T *__restrict__ P = ctrl + static_cast<size_t>(o) * DIM * NCP;
    for (int64_t j0 = 0; j0 < n_per; j0 += 64 * kPtsQ) {
        float Bu[kPtsQ][DU + 1], Bv[kPtsQ][DV + 1], Bw[kPtsQ][DW + 1];
        int64_t q[kPtsQ];
        bool ok[kPtsQ];
#pragma unroll
        for (int s = 0; s < kPtsQ; ++s) {
            const int64_t j = j0 + s * 64 + lane;
            ok[s] = j < n_per;
            q[s] = (o0 + o) * n_per + (ok[s] ? j : n_per - 1);
            const float *__restrict__ p = uvw + q[s] * NPAR;
            basis_at<DU, BASIS>(p[0], Bu[s]);
            basis_at<DV, BASIS>(p[1], Bv[s]);
            if constexpr (DW > 0) basis_at<DW, BASIS>(p[2], Bw[s]);
            else Bw[s][0] = 1.0f;
        }
        // One (coordinate, i) slab of (DV+1)(DW+1) coefficients at a time: the
        // slab loop is not unrolled, so the scalar loads of one slab are in
        // flight while the previous slab's FMAs run, and the coefficients never
        // outnumber the scalar registers (a fully unrolled nest would hoist all
        // DIM * NCP loads and spill them into vector-register lanes).
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            float acc[kPtsQ] = {};
#pragma unroll 1
            for (int i = 0; i <= DU; ++i) {
                float Ri[kPtsQ] = {};
#pragma unroll
                for (int jj = 0; jj <= DV; ++jj) {
                    float Qj[kPtsQ] = {};
#pragma unroll
                    for (int k = 0; k <= DW; ++k) {
                        const float pv = to_f32<T>(P[c * NCP + (i * (DV + 1) + jj) * (DW + 1) + k]);
#pragma unroll
                        for (int s = 0; s < kPtsQ; ++s) Qj[s] = __builtin_fmaf(Bw[s][k], pv, Qj[s]);
                    }
#pragma unroll
                    for (int s = 0; s < kPtsQ; ++s) Ri[s] = __builtin_fmaf(Bv[s][jj], Qj[s], Ri[s]);
                }
#pragma unroll
                for (int s = 0; s < kPtsQ; ++s) acc[s] = __builtin_fmaf(Bu[s][i], Ri[s], acc[s]);
            }
#pragma unroll
            for (int s = 0; s < kPtsQ; ++s)
                if (ok[s]) st_stream(out + c * plane + q[s], acc[s]);
        }
    }
}

// ------------------------------------------------------------------ MFMA grid

// ------------------------------------------------------------------ dispatch (over degrees and dim)
template <typename T, int BASIS, int DU, int DV, int DIM>
void launch_grid3(const void *ctrl, int nu, int nv, float *out, int64_t plane, int64_t o0, uint32_t n_obj,
                  hipStream_t s) {
    GridArgs g = grid_args<DU, DIM>(nu, nv, n_obj, plane);
    const size_t lds = sizeof(float) * grid_floats<DU, DIM>(g);
    const int64_t npts = static_cast<int64_t>(nu) * nv;
    // at most 2^30 points and 2^23 workgroups per launch (a patch has at most 2^24 points)
    const int64_t per = g.per_strip == 0 ? (int64_t(1) << 30) / npts
                                         : std::max<int64_t>(1, (int64_t(1) << 23) / (static_cast<int64_t>(g.per_strip) * g.strips));
    for (int64_t p0 = 0; p0 < n_obj; p0 += per) {
        const int64_t np = std::min<int64_t>(per, n_obj - p0);
        if (g.per_strip == 0) g.n = static_cast<uint32_t>(np * npts);
        g.o0 = o0 + p0;
        const int64_t blocks = g.per_strip == 0 ? (np * npts + 31 + g.chunk - 1) / g.chunk : np * g.per_strip * g.strips;
        hipLaunchKernelGGL((k_tensor_grid<DU, DV, DIM, T, BASIS>), dim3(static_cast<uint32_t>(blocks)), dim3(kBlock),
                           lds, s, static_cast<const T *>(ctrl) + p0 * DIM * (DU + 1) * (DV + 1), g, out);
    }
}

template <typename T, int BASIS, int DU, int DV>
int launch_grid2(int dim, const void *ctrl, int nu, int nv, float *out, int64_t plane, int64_t o0, uint32_t blocks,
                 hipStream_t s) {
    switch (dim) {
        case 1: launch_grid3<T, BASIS, DU, DV, 1>(ctrl, nu, nv, out, plane, o0, blocks, s); break;
        case 2: launch_grid3<T, BASIS, DU, DV, 2>(ctrl, nu, nv, out, plane, o0, blocks, s); break;
        case 3: launch_grid3<T, BASIS, DU, DV, 3>(ctrl, nu, nv, out, plane, o0, blocks, s); break;
        default: launch_grid3<T, BASIS, DU, DV, 4>(ctrl, nu, nv, out, plane, o0, blocks, s); break;
    }
    return BZ_OK;
}

template <typename T, int BASIS, int DU>
int launch_grid1(int dv, int dim, const void *ctrl, int nu, int nv, float *out, int64_t plane, int64_t o0,
                 uint32_t blocks, hipStream_t s) {
    switch (dv) {
        case 1: return launch_grid2<T, BASIS, DU, 1>(dim, ctrl, nu, nv, out, plane, o0, blocks, s);
        case 2: return launch_grid2<T, BASIS, DU, 2>(dim, ctrl, nu, nv, out, plane, o0, blocks, s);
        case 3: return launch_grid2<T, BASIS, DU, 3>(dim, ctrl, nu, nv, out, plane, o0, blocks, s);
        default: return launch_grid2<T, BASIS, DU, 4>(dim, ctrl, nu, nv, out, plane, o0, blocks, s);
    }
}

template <typename T, int BASIS>
int launch_grid(int du, int dv, int dim, const void *ctrl, int nu, int nv, float *out, int64_t plane, int64_t o0,
                uint32_t blocks, hipStream_t s) {
    switch (du) {
        case 1: return launch_grid1<T, BASIS, 1>(dv, dim, ctrl, nu, nv, out, plane, o0, blocks, s);
        case 2: return launch_grid1<T, BASIS, 2>(dv, dim, ctrl, nu, nv, out, plane, o0, blocks, s);
        case 3: return launch_grid1<T, BASIS, 3>(dv, dim, ctrl, nu, nv, out, plane, o0, blocks, s);
        default: return launch_grid1<T, BASIS, 4>(dv, dim, ctrl, nu, nv, out, plane, o0, blocks, s);
    }
}

template <typename T, int BASIS, int DU, int DV, int DW>
int launch_pts3(int dim, const void *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane, int64_t o0,
                uint32_t n_obj, hipStream_t s) {
    const T *p = static_cast<const T *>(ctrl);
    const uint32_t blocks = (n_obj + kBlock / 64 - 1) / (kBlock / 64);
    switch (dim) {
        case 1: hipLaunchKernelGGL((k_tensor_points<DU, DV, DW, 1, T, BASIS>), dim3(blocks), dim3(kBlock), 0, s, p, uvw, n_per, n_obj, out, plane, o0); break;
        case 2: hipLaunchKernelGGL((k_tensor_points<DU, DV, DW, 2, T, BASIS>), dim3(blocks), dim3(kBlock), 0, s, p, uvw, n_per, n_obj, out, plane, o0); break;
        case 3: hipLaunchKernelGGL((k_tensor_points<DU, DV, DW, 3, T, BASIS>), dim3(blocks), dim3(kBlock), 0, s, p, uvw, n_per, n_obj, out, plane, o0); break;
        default: hipLaunchKernelGGL((k_tensor_points<DU, DV, DW, 4, T, BASIS>), dim3(blocks), dim3(kBlock), 0, s, p, uvw, n_per, n_obj, out, plane, o0); break;
    }
    return BZ_OK;
}

template <typename T, int BASIS, int DU, int DV>
int launch_pts2(int dw, int dim, const void *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane,
                int64_t o0, uint32_t blocks, hipStream_t s) {
    switch (dw) {
        case 0: return launch_pts3<T, BASIS, DU, DV, 0>(dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 1: return launch_pts3<T, BASIS, DU, DV, 1>(dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 2: return launch_pts3<T, BASIS, DU, DV, 2>(dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 3: return launch_pts3<T, BASIS, DU, DV, 3>(dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        default: return launch_pts3<T, BASIS, DU, DV, 4>(dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
    }
}

template <typename T, int BASIS, int DU>
int launch_pts1(int dv, int dw, int dim, const void *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane,
                int64_t o0, uint32_t blocks, hipStream_t s) {
    switch (dv) {
        case 1: return launch_pts2<T, BASIS, DU, 1>(dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 2: return launch_pts2<T, BASIS, DU, 2>(dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 3: return launch_pts2<T, BASIS, DU, 3>(dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        default: return launch_pts2<T, BASIS, DU, 4>(dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
    }
}

template <typename T, int BASIS>
int launch_pts(int du, int dv, int dw, int dim, const void *ctrl, const float *uvw, int64_t n_per, float *out,
               int64_t plane, int64_t o0, uint32_t blocks, hipStream_t s) {
    switch (du) {
        case 1: return launch_pts1<T, BASIS, 1>(dv, dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 2: return launch_pts1<T, BASIS, 2>(dv, dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        case 3: return launch_pts1<T, BASIS, 3>(dv, dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
        default: return launch_pts1<T, BASIS, 4>(dv, dw, dim, ctrl, uvw, n_per, out, plane, o0, blocks, s);
    }
}

}  // namespace
}  // namespace bzi
