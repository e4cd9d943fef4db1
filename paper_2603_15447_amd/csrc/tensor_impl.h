// Separable tensor-product kernels shared by the Bernstein (tensor.hip) and
// per-axis Seiler (tensor_seiler.hip) evaluators of surfaces and volumes
// (Sec. 2.2: the order splits over the parameter axes).  The contraction is
// the same for both; only the per-axis basis differs.
//
//  k_tensor_grid   nu x nv uniform grids: a workgroup contracts the net with
//                  the v basis once per grid column (isoline coefficients
//                  R_i(v_b), shared through LDS with the u basis of its rows),
//                  then du+1 FMAs per coordinate and point.
//  k_tensor_grid_patch  calls of few patches, rows or long columns: a patch per
//                  workgroup.
//  k_tensor_points_staged  surfaces at random (u,v) per query: a run of queries
//                  per workgroup, their objects' nets in LDS, v -> u per lane.
//  k_tensor_points one object per wavefront, random (u,v,w) per query, 4
//                  queries per lane, separable contraction w -> v -> u.
//  k_tensor_points_mfma  volumes of degrees 2 and 3 likewise, w contracted on the
//                  matrix cores.
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

// One patch per workgroup, without tables of the columns (grid_by_patch says
// where): where nv divides the block size every thread keeps one grid column b,
// contracts the net with the v basis once (isoline coefficients R_i(v_b)) and
// evaluates its points of that column with the u basis of their rows, from a
// table in LDS when nu <= block size; else every point on its own.  NU, NV > 0 fix
// the grid size at compile time: the row loop unrolls, with du = dv the column
// basis is a row of the same table, and each column is contracted once, by one
// thread, and shared with the other threads of that column through LDS; 0 takes
// nu, nv at run time.  The same basis at the same parameters a/(nu-1), b/(nv-1) as
// k_tensor_grid, in the same order: the same bits.
template <int DU, int DV, int DIM, typename T, int BASIS, int NU, int NV>
__device__ __forceinline__ void grid_columns(const T *__restrict__ P, int nu_rt, int nv_rt, float du_den, float dv_den,
                                             float *__restrict__ ob, int64_t plane, float *tab_u) {
    constexpr int NCP = (DU + 1) * (DV + 1);
    const int nu = NU > 0 ? NU : nu_rt;
    const int nv = NV > 0 ? NV : nv_rt;
    const int b = threadIdx.x % nv;
    const int a0 = threadIdx.x / nv;
    const int astep = kBlock / nv;
    const bool table = nu <= kBlock;
    if (table) {
        if (static_cast<int>(threadIdx.x) < nu) {
            float Bu[DU + 1];
            basis_at<DU, BASIS>(static_cast<float>(threadIdx.x) / du_den, Bu);
#pragma unroll
            for (int i = 0; i <= DU; ++i) tab_u[threadIdx.x * (DU + 1) + i] = Bu[i];
        }
        __syncthreads();
    }
    // isoline coefficients of column b: R[c][i] = sum_j Bv_j(b) P[c][i][j]
    auto contract = [&](float (&R)[DIM][DU + 1]) {
        float Bv[DV + 1];
        if constexpr (NU > 0 && NU == NV && DU == DV) {
#pragma unroll
            for (int j = 0; j <= DV; ++j) Bv[j] = tab_u[b * (DU + 1) + j];
        } else {
            basis_at<DV, BASIS>(static_cast<float>(b) / dv_den, Bv);
        }
#pragma unroll
        for (int c = 0; c < DIM; ++c)
#pragma unroll
            for (int i = 0; i <= DU; ++i) {
                float acc = Bv[0] * to_f32<T>(P[c * NCP + i * (DV + 1)]);
#pragma unroll
                for (int j = 1; j <= DV; ++j)
                    acc = __builtin_fmaf(Bv[j], to_f32<T>(P[c * NCP + i * (DV + 1) + j]), acc);
                R[c][i] = acc;
            }
    };
    float R[DIM][DU + 1];
    if constexpr (NU > 0) {
        static_assert(NU <= kBlock && NU % (kBlock / NV) == 0, "fixed grids fill whole row steps");
        // the first NV threads contract one column each; the kBlock / NV
        // threads of a column share it through LDS
        __shared__ __align__(16) float tab_r[NV * DIM * (DU + 1)];
        if (static_cast<int>(threadIdx.x) < NV) {
            float Rc[DIM][DU + 1];
            contract(Rc);
#pragma unroll
            for (int c = 0; c < DIM; ++c)
#pragma unroll
                for (int i = 0; i <= DU; ++i) tab_r[(b * DIM + c) * (DU + 1) + i] = Rc[c][i];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < DIM; ++c)
#pragma unroll
            for (int i = 0; i <= DU; ++i) R[c][i] = tab_r[(b * DIM + c) * (DU + 1) + i];
        const uint32_t lo = static_cast<uint32_t>(a0 * NV + b);
#pragma unroll
        for (int k = 0; k < NU / (kBlock / NV); ++k) {
            const int a = a0 + k * (kBlock / NV);
            float Bu[DU + 1];
#pragma unroll
            for (int i = 0; i <= DU; ++i) Bu[i] = tab_u[a * (DU + 1) + i];
#pragma unroll
            for (int c = 0; c < DIM; ++c) st_stream(ob + c * plane + (lo + k * kBlock), dot_basis<DU>(Bu, R[c]));
        }
        return;
    }
    contract(R);
    float *__restrict__ oc = ob + a0 * nv + b;
    if (table) {
        for (int a = a0; a < nu; a += astep, oc += kBlock) {
            float Bu[DU + 1];
#pragma unroll
            for (int i = 0; i <= DU; ++i) Bu[i] = tab_u[a * (DU + 1) + i];
#pragma unroll
            for (int c = 0; c < DIM; ++c) st_stream(oc + c * plane, dot_basis<DU>(Bu, R[c]));
        }
    } else {
        for (int a = a0; a < nu; a += astep, oc += kBlock) {
            float Bu[DU + 1];
            basis_at<DU, BASIS>(static_cast<float>(a) / du_den, Bu);
#pragma unroll
            for (int c = 0; c < DIM; ++c) st_stream(oc + c * plane, dot_basis<DU>(Bu, R[c]));
        }
    }
}

template <int DU, int DV, int DIM, typename T, int BASIS>
__global__ __launch_bounds__(kBlock) void k_tensor_grid_patch(const T *__restrict__ ctrl, int nu, int nv,
                                                        float *__restrict__ out, int64_t plane, int64_t o0) {
    constexpr int NCP = (DU + 1) * (DV + 1);
    const uint32_t o = blockIdx.x;
    const T *__restrict__ P = ctrl + static_cast<size_t>(o) * DIM * NCP;
    const int npts = nu * nv;
    float *__restrict__ ob = out + (o0 + o) * static_cast<int64_t>(npts);
    const float du_den = nu > 1 ? static_cast<float>(nu - 1) : 1.0f;
    const float dv_den = nv > 1 ? static_cast<float>(nv - 1) : 1.0f;
    __shared__ __align__(16) float tab_u[kBlock * (DU + 1)];
    if (kBlock % nv == 0) {
        if (nu == 32 && nv == 32) grid_columns<DU, DV, DIM, T, BASIS, 32, 32>(P, nu, nv, du_den, dv_den, ob, plane, tab_u);
        else grid_columns<DU, DV, DIM, T, BASIS, 0, 0>(P, nu, nv, du_den, dv_den, ob, plane, tab_u);
    } else {
        for (int p = threadIdx.x; p < npts; p += kBlock) {
            const int a = p / nv, b = p - (p / nv) * nv;
            float Bu[DU + 1], Bv[DV + 1];
            basis_at<DU, BASIS>(static_cast<float>(a) / du_den, Bu);
            basis_at<DV, BASIS>(static_cast<float>(b) / dv_den, Bv);
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                float Ri[DU + 1];
#pragma unroll
                for (int i = 0; i <= DU; ++i) {
                    float acc = Bv[0] * to_f32<T>(P[c * NCP + i * (DV + 1)]);
#pragma unroll
                    for (int j = 1; j <= DV; ++j)
                        acc = __builtin_fmaf(Bv[j], to_f32<T>(P[c * NCP + i * (DV + 1) + j]), acc);
                    Ri[i] = acc;
                }
                st_stream(ob + c * plane + p, dot_basis<DU>(Bu, Ri));
            }
        }
    }
}

// ------------------------------------------------------------------ VALU points
// Volumes, one object per wavefront, 4 queries per lane at a time: the object's
// control points are wave-uniform (scalar loads into SGPRs) and each one
// feeds the FMAs of 4 queries.  Separable contraction w -> v -> u.  An
// object's queries go to waves_per_obj wavefronts, of per_wave * 64 * kPtsQ each.
constexpr int kPtsQ = 4;

template <int DU, int DV, int DW, int DIM, typename T, int BASIS>
__global__ __launch_bounds__(kBlock) void k_tensor_points(const T *__restrict__ ctrl, const float *__restrict__ uvw,
                                                          int64_t n_per, uint32_t n_obj, uint32_t waves_per_obj,
                                                          int per_wave, float *__restrict__ out, int64_t plane,
                                                          int64_t o0) {
    constexpr int NCP = (DU + 1) * (DV + 1) * (DW + 1);
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6));
    uint32_t o = w, part = 0;
    if (waves_per_obj > 1) {  // (the division is a good part of what a small object takes)
        o = w / waves_per_obj;
        part = w - o * waves_per_obj;
    }
    if (o >= n_obj) return;
    const int lane = threadIdx.x & 63;
    const T *__restrict__ P = ctrl + static_cast<size_t>(o) * DIM * NCP;
    const int64_t j_begin = static_cast<int64_t>(part) * per_wave * (64 * kPtsQ);
    const int64_t j_end = min(n_per, j_begin + static_cast<int64_t>(per_wave) * (64 * kPtsQ));
    for (int64_t j0 = j_begin; j0 < j_end; j0 += 64 * kPtsQ) {
        float Bu[kPtsQ][DU + 1], Bv[kPtsQ][DV + 1], Bw[kPtsQ][DW + 1];
        int64_t q[kPtsQ];
        bool ok[kPtsQ];
#pragma unroll
        for (int s = 0; s < kPtsQ; ++s) {
            const int64_t j = j0 + s * 64 + lane;
            ok[s] = j < n_per;
            q[s] = (o0 + o) * n_per + (ok[s] ? j : n_per - 1);
            const float *__restrict__ p = uvw + q[s] * 3;
            basis_at<DU, BASIS>(p[0], Bu[s]);
            basis_at<DV, BASIS>(p[1], Bv[s]);
            basis_at<DW, BASIS>(p[2], Bw[s]);
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

// ------------------------------------------------------------------ staged points
// Surfaces: a workgroup takes a run of `chunk` queries, whichever objects they
// belong to, and stages those objects' nets in LDS; each lane then reads its own
// object's net (a wavefront's lanes share few objects, whose reads are
// broadcasts) and contracts v and u, in k_tensor_points' order.  Points of
// misaligned planes go through LDS to be stored as whole lines, as in
// k_curves_mixed.
// Bound by the 20 bytes per query and by the LDS reads of the net (12 of 16
// bytes for a bicubic in 3D).  A wavefront per object left its lanes idle below
// 256 points and paid a chain of scalar loads per object; a single large object
// was one wavefront's.  2^22 points of 3D bicubics, wavefront per object -> staged:
// 32 points each 71-91 -> 19.6 us, 64 38-42 -> 17.1, 100 28 -> 19, 256 16.1 -> 14.8
// (5.7 TB/s), 333 21 -> 16.7, 1000 17-20 -> 15.2, 1 each 2235 -> 167.
struct PtsArgs {
    int64_t q0;     // the first query's place in uvw and in a plane
    int64_t plane;
    uint32_t nq;
    int chunk;      // queries per workgroup
    int slots;      // objects it may touch
    bool same;      // whether the planes' lines begin at the same queries
    FastDiv div_n;  // queries per object
};

template <int DU, int DV, int DIM>
struct PtsGeom {
    static constexpr int NCP = (DU + 1) * (DV + 1);
    static constexpr int PAD = (NCP + 3) / 4 * 4;  // floats per coordinate: whole 16-byte vectors
    static constexpr int OBJ = DIM * PAD + 4;      // (+ 4: neighbouring objects in other banks)
};

template <int DU, int DV, int DIM, typename T, int BASIS>
__global__ __launch_bounds__(kBlock) void k_tensor_points_staged(const T *__restrict__ ctrl, const float *__restrict__ uvw,
                                                                 PtsArgs a, float *__restrict__ out) {
    using G = PtsGeom<DU, DV, DIM>;
    constexpr int NCP = G::NCP, PAD = G::PAD;
    extern __shared__ __align__(16) float lds[];
    out += a.q0;
    const uint32_t at = blockIdx.x * a.chunk;
    const uint32_t sh = a.same ? line_offset(out) : 31u;
    const uint32_t first = at > sh ? at - sh : 0;
    const uint32_t end = min(a.nq, at + a.chunk - (a.same ? sh : 0u));
    const int n = static_cast<int>(end - first);
    if (n <= 0) return;
    const uint32_t o_lo = fdiv(first, a.div_n), s0 = first - o_lo * a.div_n.d;
    const int n_o = static_cast<int>(fdiv(s0 + n - 1, a.div_n)) + 1;
    const float *__restrict__ uv = uvw + (a.q0 + first) * 2;
    float u_next = uv[min(static_cast<int>(threadIdx.x), n - 1) * 2];  // on its way while the nets are staged
    float v_next = uv[min(static_cast<int>(threadIdx.x), n - 1) * 2 + 1];
    const T *__restrict__ P = ctrl + static_cast<size_t>(o_lo) * DIM * NCP;
#pragma unroll 4
    for (int e = threadIdx.x; e < n_o * DIM * NCP; e += kBlock) {
        const int r = e / NCP, i = e - r * NCP;
        const int k = r / DIM, c = r - k * DIM;
        lds[k * G::OBJ + c * PAD + i] = to_f32<T>(P[e]);
    }
    __syncthreads();
    float *__restrict__ buf = lds + a.slots * G::OBJ;  // [DIM][chunk + 32] unless the planes lie alike
    const int pitch = a.chunk + 32;
    auto points = [&](auto same) {
#pragma unroll 1
        for (int p = threadIdx.x; p < n; p += kBlock) {
            float Bu[DU + 1], Bv[DV + 1];
            basis_at<DU, BASIS>(u_next, Bu);
            basis_at<DV, BASIS>(v_next, Bv);
            u_next = uv[min(p + kBlock, n - 1) * 2];
            v_next = uv[min(p + kBlock, n - 1) * 2 + 1];
            const float *__restrict__ net = lds + fdiv(s0 + p, a.div_n) * G::OBJ;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                float x[PAD];
#pragma unroll
                for (int e = 0; e < PAD; e += 4) {
                    const float4 f = *reinterpret_cast<const float4 *>(net + c * PAD + e);
                    x[e] = f.x, x[e + 1] = f.y, x[e + 2] = f.z, x[e + 3] = f.w;
                }
                float acc = 0.0f;
#pragma unroll
                for (int i = 0; i <= DU; ++i) {
                    float R = 0.0f;
#pragma unroll
                    for (int j = 0; j <= DV; ++j) R = __builtin_fmaf(Bv[j], x[i * (DV + 1) + j], R);
                    acc = __builtin_fmaf(Bu[i], R, acc);
                }
                if constexpr (decltype(same)::value) st_stream(at_lane(out + c * a.plane + first, p), acc);
                else buf[c * pitch + p] = acc;
            }
        }
    };
    if (a.same) {
        points(std::true_type{});
        return;
    }
    points(std::false_type{});
    __syncthreads();
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        float *__restrict__ oc = out + c * a.plane;
        const uint32_t sc = line_offset(oc), lo = at > sc ? 0 : sc - at;  // plane queries [at - sc + lo, ...)
        // (none in the last workgroup where the plane's end lies before its part)
        const uint32_t n_own = a.nq + sc > at ? min(static_cast<uint32_t>(a.chunk), a.nq + sc - at) : 0;
        float *__restrict__ to = oc + at - sc;
        const float *__restrict__ from = buf + c * pitch + static_cast<int>(at - sc - first);
        for (uint32_t p = threadIdx.x; p < n_own; p += kBlock)
            if (p >= lo) st_stream(at_lane(to, p), from[p]);
    }
}

// ------------------------------------------------------------------ MFMA points
// Volumes of degrees up to 3 on the FP32 matrix cores.  A wavefront takes 64
// points of one object.  Each lane forms the three bases of its own point and
// shares them through LDS; the 64 points are then four tiles of 16, and per
// tile and coordinate one 16x16x4 MFMA contracts w: rows m = 4 i + j of the net
// (A: P[c][i][j][k], held for the whole object), columns the tile's points (B:
// Bw_k).  Lane (g, n) = (l / 16, l mod 16) then holds i = g, j = 0..3 of point
// n, contracts v on the vector ALU, and the four lanes of a point are added,
// times Bu_i, while the four tiles are put side by side: two exchanges between
// half-wavefronts or rows per coordinate leave lane l with point l, so that
// every coordinate is stored as 64 consecutive floats.
// About 125 vector instructions and 12 MFMAs (32 cycles of the matrix core each)
// per 64 points, where the separable contraction on the vector ALU issues 355;
// the two hardly overlap, and both draw the clock down when launches follow one
// another.  65536 tricubics x 256: 148-157 -> 111-134 us (one card, another);
// biquadratic in u and v, cubic in w: 64 -> 60; with w linear the vector ALU is
// faster (54 against 66), so w has to be of degree 2 at least.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Bernstein basis of degree up to 3 with the rounding of 1 - t carried along:
// ds is what 1 - t lost (exactly), and s^2 takes it up.  The basis is most of a
// point's error: 0.97e-7 against 1.25e-7 of the points' norm (64-bit reference)
// for tricubic points contracted either way.
template <int D>
__device__ __forceinline__ void bernstein_basis_comp(float t, float (&B)[D + 1]) {
    const float s = 1.0f - t, ds = (1.0f - s) - t;
    if constexpr (D == 1) {
        B[0] = s;
        B[1] = t;
    } else {
        // what a loss adds; not a number where t is infinite or next to it: nothing
        // is lost there, and the basis has its infinite values
        auto add = [](float x) { return x == x ? x : 0.0f; };
        const float s2 = __builtin_fmaf(s, s, add((s + s) * ds)), t2 = t * t;
        if constexpr (D == 2) {
            const float a = 2.0f * t;
            B[0] = s2;
            B[1] = __builtin_fmaf(a, s, add(a * ds));
            B[2] = t2;
        } else {
            B[0] = s2 * s;
            B[1] = (3.0f * t) * s2;
            B[2] = (3.0f * t2) * s;
            B[3] = t2 * t;
        }
    }
}

// x, y: halves (rows) b of x exchanged with halves (rows) a of y.
__device__ __forceinline__ void swap_halves(float &x, float &y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows(float &x, float &y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
}

// Workgroup: four wavefronts of 64 points at a time, `per_wave` times; wavefront
// w of object o begins at point w * per_wave * 64 of it.
// (Four waves per SIMD asked for: with at most 256 registers per lane the compiler
// lets the MFMAs write vector registers; otherwise 48 moves per 64 points fetch
// their results from the accumulation registers, 148 against 134 us.)
template <int DU, int DV, int DW, int DIM, typename T>
__global__ __launch_bounds__(kBlock, 4) void k_tensor_points_mfma(const T *__restrict__ ctrl, const float *__restrict__ uvw,
                                                               int64_t n_per, uint32_t n_obj, uint32_t waves_per_obj,
                                                               int per_wave, float *__restrict__ out, int64_t plane,
                                                               int64_t o0) {
    constexpr int NCP = (DU + 1) * (DV + 1) * (DW + 1);
    __shared__ __align__(16) float tab[kBlock / 64][3][64][4];
    const int lane = threadIdx.x & 63, g = lane >> 4, n = lane & 15;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t w = blockIdx.x * (kBlock / 64) + wid;
    const uint32_t o = w / waves_per_obj;
    if (o >= n_obj) return;
    const int64_t j_begin = static_cast<int64_t>(w - o * waves_per_obj) * per_wave * 64;
    const int64_t j_end = min(n_per, j_begin + static_cast<int64_t>(per_wave) * 64);
    if (j_begin >= j_end) return;
    const T *__restrict__ P = ctrl + static_cast<size_t>(o) * DIM * NCP;
    float A[DIM];  // row m = n: i = n / 4, j = n mod 4; k = g
    {
        const int i = n >> 2, j = n & 3;
        const bool in = i <= DU && j <= DV && g <= DW;
        const int at = in ? (i * (DV + 1) + j) * (DW + 1) + g : 0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) A[c] = in ? to_f32<T>(P[c * NCP + at]) : 0.0f;
    }
    float (*__restrict__ tu)[4] = tab[wid][0], (*__restrict__ tv)[4] = tab[wid][1], (*__restrict__ tw)[4] = tab[wid][2];
    const int64_t q0 = (o0 + o) * n_per + j_begin;
    const int n_here = static_cast<int>(j_end - j_begin);
    // parameters of point p of the wavefront's (of its last beyond), and its
    // results, from wave-uniform bases
    const float *__restrict__ up = uvw + q0 * 3;
    float *__restrict__ ob = out + q0;
    typedef float f32x3 __attribute__((ext_vector_type(3), aligned(4)));
    auto params = [&](int p) {
        return *reinterpret_cast<const f32x3 *>(reinterpret_cast<const char *>(up) +
                                                static_cast<size_t>(12u * static_cast<uint32_t>(min(p, n_here - 1))));
    };
    f32x3 x = params(lane);
    for (int p0 = 0; p0 < n_here; p0 += 64) {
        float Bu[DU + 1], Bv[DV + 1], Bw[DW + 1];
        bernstein_basis_comp<DU>(x[0], Bu);
        bernstein_basis_comp<DV>(x[1], Bv);
        bernstein_basis_comp<DW>(x[2], Bw);
        if (p0 + 64 < n_here) x = params(p0 + 64 + lane);  // the next ones, on their way meanwhile
        auto at = [](const auto &B, int i, int d) { return i <= d ? B[i] : 0.0f; };
        // (the wavefront's own part of LDS: its instructions are in order, no barrier)
        *reinterpret_cast<f32x4 *>(tu[lane]) = f32x4{Bu[0], at(Bu, 2, DU), Bu[1], at(Bu, 3, DU)};
        *reinterpret_cast<f32x4 *>(tv[lane]) = f32x4{Bv[0], Bv[1], at(Bv, 2, DV), at(Bv, 3, DV)};
        *reinterpret_cast<f32x4 *>(tw[lane]) = f32x4{Bw[0], Bw[1], at(Bw, 2, DW), at(Bw, 3, DW)};
        __builtin_amdgcn_wave_barrier();
        float R[4][DIM];  // tile, coordinate: contracted over w and v
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float b = tw[16 * t + n][g];
            const f32x4 v = *reinterpret_cast<const f32x4 *>(tv[16 * t + n]);
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                const f32x4 q = __builtin_amdgcn_mfma_f32_16x16x4f32(A[c], b, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
                float r = v[0] * q[0];
#pragma unroll
                for (int j = 1; j <= DV; ++j) r = __builtin_fmaf(v[j], q[j], r);
                // (rows past the net are zero, but not times an infinite basis)
                R[t][c] = DU == 3 || g <= DU ? r : 0.0f;
            }
        }
        // Bu_i and Bu_(i+2), i = g mod 2, of this lane's tile of the pairs (0, 2) and (1, 3)
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const int row = 16 * (g & 2) + n, pos = 2 * (g & 1);
        const f32x2 u02 = *reinterpret_cast<const f32x2 *>(&tu[row][pos]);
        const f32x2 u13 = *reinterpret_cast<const f32x2 *>(&tu[row + 16][pos]);
        __builtin_amdgcn_wave_barrier();
        const bool ok = p0 + lane < n_here;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            swap_halves(R[0][c], R[2][c]);
            swap_halves(R[1][c], R[3][c]);
            float a = __builtin_fmaf(u02[1], R[2][c], u02[0] * R[0][c]);
            float b = __builtin_fmaf(u13[1], R[3][c], u13[0] * R[1][c]);
            swap_rows(a, b);
            if (ok) st_stream(at_lane(ob + c * plane, p0 + lane), a + b);
        }
    }
}

// ------------------------------------------------------------------ dispatch (over degrees and dim)
// Whether a grid call takes a workgroup per patch (k_tensor_grid_patch) rather
// than chunks of the output with tables (k_tensor_grid).  A patch per workgroup
// has no tables to fill before its first point, which calls of few patches and
// grids of one to three rows (a column's contraction serves no others) show; its
// stores begin where a patch begins, and small patches leave its threads idle, so
// large calls go in chunks, but for 1D points and for few rows of a nv that divides
// the block size, where a thread has one column and few points of it.  By patches,
// points, control points of a patch and floats of output, from 5,000 random calls
// of up to 2^24 points, 2,500 more of up to 2^26 with such nv and 2,500 of 1024 points
// a patch about, on rotating buffers: so chosen they take 1 % more time than with the better kernel each, all
// in chunks 6 to 8 % more (7805 patches x 32 x 32 in 1D: 6.5 us by patch, 10.7 in
// chunks; 5 patches x 8 x 31 in 4D: 2.1 and 3.0; 8417 x 1 x 191 in 3D: 8.1 and
// 21.7; 4096 x 32 x 32 in 2D 6.9 and 8.7, 65536 of them 88 and 80; 8000 x 64 x 64
// in 2D 114 and 94; 33 x 33 points of 16384 patches 75 and 35).  16-bit nets of 25
// control points are the slow ones of run-time rows by patch (2276 x 128 x 8 in 3D:
// 13.7 and 6.1).
inline bool grid_by_patch(int nu, int nv, int64_t n, int ncp, int dim, bool f32) {
    const int64_t pts = static_cast<int64_t>(nu) * nv, work = n * pts * ncp, floats = n * pts * dim;
    if (nu == 32 && nv == 32) return dim == 1 || floats < 1 << 24;
    if (nu <= (f32 ? 3 : 2) && dim > 1 && pts < 2048 && pts >= (nu == 1 ? 64 : 256)) return true;
    if (kBlock % nv == 0) {
        if (!f32 && ncp >= 25 && nv <= 64) return false;
        if (pts >= 1024)
            return n >= (pts >= 2048 ? 256 : 128) && (dim == 1 || nu < 16 || floats < 1 << (pts >= 2048 ? 23 : 24));
        return n < (pts >= 256 ? 1024 : 256) || (nu >= 4 && nv >= 128);
    }
    if (pts >= 2048) return false;
    if (pts >= 1024) return dim > 1 && ncp < (f32 ? 20 : 15) && (n == 1 || (n >= 96 && work < 1 << 22));
    return n < 2048 && work < (f32 ? 1 << 22 : 1 << 21);
}

template <typename T, int BASIS, int DU, int DV, int DIM>
void launch_grid3(const void *ctrl, int nu, int nv, float *out, int64_t plane, int64_t o0, uint32_t n_obj,
                  hipStream_t s) {
    if (grid_by_patch(nu, nv, n_obj, (DU + 1) * (DV + 1), DIM, std::is_same<T, float>::value)) {
        hipLaunchKernelGGL((k_tensor_grid_patch<DU, DV, DIM, T, BASIS>), dim3(n_obj), dim3(kBlock), 0, s,
                           static_cast<const T *>(ctrl), nu, nv, out, plane, o0);
        return;
    }
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

// Which kernel (see k_tensor_points_mfma).
template <int BASIS, int DU, int DV, int DW>
constexpr bool kPointsMfma = BASIS == kBasisBernstein && DW >= 2 && DU <= 3 && DV <= 3 && DW <= 3 &&
                             (DU + 1) * (DV + 1) * (DW + 1) >= 27;

// Surfaces' points: chunks of 1024 queries, fewer in calls too small to give
// every CU two workgroups and where the nets of so many would not leave a CU
// four; 128 queries' nets fit a workgroup's 64 KB at any degree, even with one
// point each.  At most 2^30 queries per launch: whole objects, or pieces of one.
template <typename T, int BASIS, int DU, int DV, int DIM>
void launch_pts_staged(const T *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane, int64_t o0,
                       int64_t n_obj, hipStream_t s) {
    using G = PtsGeom<DU, DV, DIM>;
    static_assert(128 * G::OBJ <= 16384 && 127 * G::OBJ + DIM * 128 <= 16384, "128 queries' nets fit 64 KB");
    constexpr int64_t kMost = int64_t(1) << 30;
    const int64_t per = std::min(n_per, kMost), step = kMost / per;
    PtsArgs a;
    a.plane = plane;
    a.same = DIM == 1 || plane % 16 == 0;
    for (int64_t i = 0; i < n_obj; i += step)
        for (int64_t j = 0; j < n_per; j += per) {
            const int64_t piece = std::min(per, n_per - j);
            a.q0 = (o0 + i) * n_per + j;
            a.nq = static_cast<uint32_t>(std::min(step, n_obj - i) * piece);
            a.div_n = make_fastdiv(static_cast<uint32_t>(piece));
            size_t floats = 0;
            for (int want = a.nq >= 1024u * 512 ? 1024 : a.nq >= 512u * 512 ? 512 : 256;; want /= 2) {
                a.chunk = a.same ? want : want - 32;  // with the planes' own first queries: whole threads
                const int64_t span = a.chunk + (a.same ? 0 : 31);
                a.slots = static_cast<int>((span + piece - 2) / piece + 1);
                floats = static_cast<size_t>(a.slots) * G::OBJ + (a.same ? 0 : DIM * (a.chunk + 32));
                if (floats <= 10240 || want == 128) break;
            }
            const uint32_t blocks = (a.nq + 31 + a.chunk - 1) / a.chunk;
            hipLaunchKernelGGL((k_tensor_points_staged<DU, DV, DIM, T, BASIS>), dim3(blocks), dim3(kBlock),
                               floats * sizeof(float), s, ctrl + i * DIM * G::NCP, uvw, a, out);
        }
}

template <typename T, int BASIS, int DU, int DV, int DW, int DIM>
void launch_pts4(const T *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane, int64_t o0,
                 uint32_t n_obj, hipStream_t s) {
    constexpr bool MFMA = kPointsMfma<BASIS, DU, DV, DW>;
    // pieces of an object's queries, 64 times the queries per lane; up to 4 x 64
    // queries per wavefront while that leaves 16 wavefronts per CU (626 tricubics
    // x 604: 12.5 us with a wavefront per object, 6.2 so)
    const int q = MFMA ? 1 : kPtsQ;
    const int64_t pieces = (n_per + 64 * q - 1) / (64 * q);
    const int64_t most = MFMA ? 4 : 1;
    const int64_t per = std::max<int64_t>({1, std::min({most, pieces, n_obj * pieces / 4096}), (pieces + (1 << 20)) >> 21});
    const uint32_t wpo = static_cast<uint32_t>((pieces + per - 1) / per);
    // at most 2^25 wavefronts per launch
    const int64_t step = std::max<int64_t>(1, (int64_t(1) << 25) / wpo);
    for (int64_t i = 0; i < n_obj; i += step) {
        const uint32_t no = static_cast<uint32_t>(std::min<int64_t>(step, n_obj - i));
        const uint64_t waves = static_cast<uint64_t>(no) * wpo;
        const dim3 blocks(static_cast<uint32_t>((waves + kBlock / 64 - 1) / (kBlock / 64)));
        const T *p = ctrl + i * DIM * (DU + 1) * (DV + 1) * (DW + 1);
        const int pw = static_cast<int>(per);
        if constexpr (MFMA)
            hipLaunchKernelGGL((k_tensor_points_mfma<DU, DV, DW, DIM, T>), blocks, dim3(kBlock), 0, s, p, uvw, n_per, no,
                               wpo, pw, out, plane, o0 + i);
        else
            hipLaunchKernelGGL((k_tensor_points<DU, DV, DW, DIM, T, BASIS>), blocks, dim3(kBlock), 0, s, p, uvw, n_per,
                               no, wpo, pw, out, plane, o0 + i);
    }
}

template <typename T, int BASIS, int DU, int DV, int DW, int DIM>
void launch_pts_dim(const T *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane, int64_t o0,
                    uint32_t n_obj, hipStream_t s) {
    if constexpr (DW == 0) launch_pts_staged<T, BASIS, DU, DV, DIM>(ctrl, uvw, n_per, out, plane, o0, n_obj, s);
    else launch_pts4<T, BASIS, DU, DV, DW, DIM>(ctrl, uvw, n_per, out, plane, o0, n_obj, s);
}

template <typename T, int BASIS, int DU, int DV, int DW>
int launch_pts3(int dim, const void *ctrl, const float *uvw, int64_t n_per, float *out, int64_t plane, int64_t o0,
                uint32_t n_obj, hipStream_t s) {
    const T *p = static_cast<const T *>(ctrl);
    switch (dim) {
        case 1: launch_pts_dim<T, BASIS, DU, DV, DW, 1>(p, uvw, n_per, out, plane, o0, n_obj, s); break;
        case 2: launch_pts_dim<T, BASIS, DU, DV, DW, 2>(p, uvw, n_per, out, plane, o0, n_obj, s); break;
        case 3: launch_pts_dim<T, BASIS, DU, DV, DW, 3>(p, uvw, n_per, out, plane, o0, n_obj, s); break;
        default: launch_pts_dim<T, BASIS, DU, DV, DW, 4>(p, uvw, n_per, out, plane, o0, n_obj, s); break;
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
