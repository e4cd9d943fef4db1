// Curve evaluation kernels (integral and rational Bezier curves) for gfx950.
//
// Query q = c*n_t + j is one (curve, parameter) pair; the evaluation form is
// unrolled at compile time for each degree 1..15 and dimension 1..4, and
// results go out with non-temporal stores to the planar out[dim][n*n_t].
//  k_curves        one query per thread, its curve's control points loaded for
//                  it: by scalar loads where a wavefront stays on one curve.
//  k_curves_mixed  a workgroup stages the control points of its curves in LDS,
//                  ready for the form.
#pragma once

#include "common.h"

namespace bzi {

enum Form { FORM_DC = 0, FORM_BERN = 1, FORM_SEILER = 2, FORM_SEILER_PRE = 3 };

// ---------------------------------------------------------------- forms
// de Casteljau (Sec. 2): d levels of lerps with the same t.
template <int D>
__device__ __forceinline__ float eval_dc(const float (&b)[D + 1], float t) {
    float p[D + 1];
#pragma unroll
    for (int i = 0; i <= D; ++i) p[i] = b[i];
#pragma unroll
    for (int lvl = 1; lvl <= D; ++lvl)
#pragma unroll
        for (int i = 0; i <= D - lvl; ++i) p[i] = lerp(p[i], p[i + 1], t);
    return p[0];
}

// Bernstein basis B_{i,D}(t) = C(D,i) t^i (1-t)^(D-i); exact 1/0 at the ends.
template <int D>
__device__ __forceinline__ void bernstein_basis(float t, float (&B)[D + 1]) {
    const float s = 1.0f - t;
    float tp[D + 1], sp[D + 1];
    tp[0] = 1.0f;
    sp[0] = 1.0f;
#pragma unroll
    for (int i = 1; i <= D; ++i) {
        tp[i] = tp[i - 1] * t;
        sp[i] = sp[i - 1] * s;
    }
#pragma unroll
    for (int i = 0; i <= D; ++i) B[i] = (binomf(D, i) * tp[i]) * sp[D - i];
}

template <int D>
__device__ __forceinline__ float dot_basis(const float (&B)[D + 1], const float (&b)[D + 1]) {
    float acc = B[0] * b[0];
#pragma unroll
    for (int i = 1; i <= D; ++i) acc = __builtin_fmaf(B[i], b[i], acc);
    return acc;
}

// Seiler difference terms by peeling (Sec. 3.1): Q - L(Q_0,Q_n,t) = st Q'
// with Q'_{i-1} = (Q_i - ((n-i)/n)Q_0 - (i/n)Q_n) * n(n-1)/(i(n-i)).
// Output order [b0, bd, d1, d_{d-1}, d2, d_{d-2}, ...].  The terms grow like
// C(d, d/2) and peeling cancels; the stand-alone conversion works in FP64
// (Acc = double) and rounds each term once.  Evaluations that derive the terms
// on the fly peel in FP32 at every degree: the evaluation multiplies term i by
// (st)^i <= 4^-i, which shrinks the peeling error of the large middle terms
// as much as it grows, so FP32 peeling ends within the error of FP64 peeling
// followed by the same FP32 evaluation (a few 1e-6 of the box at degree 15).
__device__ __forceinline__ float fma_acc(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_acc(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <int D, typename Acc = double, typename Out = float, typename In = float>
__device__ __forceinline__ void seiler_terms(const In (&b)[D + 1], Out (&sc)[D + 1]) {
    Acc Q[D + 1];
#pragma unroll
    for (int i = 0; i <= D; ++i) Q[i] = static_cast<Acc>(b[i]);
    sc[0] = static_cast<Out>(b[0]);
    sc[1] = static_cast<Out>(b[D]);
    int pos = 2;
#pragma unroll
    for (int n = D; n >= 2; n -= 2) {
        Acc R[D + 1];
#pragma unroll
        for (int i = 1; i <= n - 1; ++i) {
            const Acc a0 = static_cast<Acc>(n - i) / static_cast<Acc>(n);
            const Acc a1 = static_cast<Acc>(i) / static_cast<Acc>(n);
            const Acc sc_f = static_cast<Acc>(n * (n - 1)) / static_cast<Acc>(i * (n - i));
            const Acc r = Q[i] - fma_acc(a0, Q[0], a1 * Q[n]);
            R[i - 1] = r * sc_f;
        }
#pragma unroll
        for (int i = 0; i <= n - 2; ++i) Q[i] = R[i];
        sc[pos++] = static_cast<Out>(Q[0]);
        if (n - 2 > 0) sc[pos++] = static_cast<Out>(Q[n - 2]);
    }
}

// FP32 Seiler terms of the products P_i w_i: the inner ones enter the first
// peeling unrounded (one FMA each), which the rational points' error shows
// (cubics: 3.95e-8 of the points' norm, 4.03e-8 from rounded products).
template <int D>
__device__ __forceinline__ void seiler_terms_of_products(const float (&P)[D + 1], const float (&w)[D + 1], float (&sc)[D + 1]) {
    sc[0] = P[0] * w[0];
    sc[1] = P[D] * w[D];
    if constexpr (D >= 2) {
        float R[D - 1];
#pragma unroll
        for (int i = 1; i <= D - 1; ++i) {
            const float a0 = static_cast<float>(D - i) / static_cast<float>(D), a1 = static_cast<float>(i) / static_cast<float>(D);
            const float sc_f = static_cast<float>(D * (D - 1)) / static_cast<float>(i * (D - i));
            R[i - 1] = __builtin_fmaf(P[i], w[i], -__builtin_fmaf(a0, sc[0], a1 * sc[1])) * sc_f;
        }
        if constexpr (D <= 3) {
#pragma unroll
            for (int i = 0; i < D - 1; ++i) sc[2 + i] = R[i];
        } else {
            float in[D - 1];
            seiler_terms<D - 2, float>(R, in);
#pragma unroll
            for (int i = 0; i < D - 1; ++i) sc[2 + i] = in[i];
        }
    }
}

// Seiler evaluation (Sec. 3.1), innermost level first:
// D = d_{d/2} (even d) or 0; D = L(d_i, d_{d-i}, t) + st D; C = L(b0,bd,t) + st D.
template <int D>
__device__ __forceinline__ float eval_seiler(const float (&sc)[D + 1], float t, float st) {
    constexpr int NP = (D - 1) / 2;
    float acc = (D % 2 == 0) ? sc[2 + 2 * NP] : 0.0f;
#pragma unroll
    for (int i = NP; i >= 1; --i) acc = __builtin_fmaf(st, acc, lerp(sc[2 * i], sc[2 * i + 1], t));
    return __builtin_fmaf(st, acc, lerp(sc[0], sc[1], t));
}

// Evaluate CH channels of degree-D data with form F.
template <int D, int CH, int F>
__device__ __forceinline__ void eval_channels(const float (&b)[CH][D + 1], float t, float (&r)[CH]) {
    if constexpr (F == FORM_DC) {
#pragma unroll
        for (int k = 0; k < CH; ++k) r[k] = eval_dc<D>(b[k], t);
    } else if constexpr (F == FORM_BERN) {
        float B[D + 1];
        bernstein_basis<D>(t, B);
#pragma unroll
        for (int k = 0; k < CH; ++k) r[k] = dot_basis<D>(B, b[k]);
    } else {
        const float st = (1.0f - t) * t;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            if constexpr (F == FORM_SEILER) {
                float sc[D + 1];
                seiler_terms<D, float>(b[k], sc);
                r[k] = eval_seiler<D>(sc, t, st);
            } else {
                r[k] = eval_seiler<D>(b[k], t, st);
            }
        }
    }
}

// FP64 de Casteljau on homogeneous points, used to re-evaluate rational
// points whose weight sum is ill-conditioned in FP32.  Inlined where it is
// used, once per kernel, and evaluating one row at a time: as a function of its
// own, its registers and the call's held every rational kernel at five waves per
// SIMD.  AHEAD: the next row is on its way meanwhile, and the weights are held
// (calls with signed weights of up to 2^17 queries take 0.83 of the time without).
template <int D, int DIM, bool AHEAD, typename T>
__device__ __forceinline__ void rational_fp64(const T *__restrict__ ctrl, const T *__restrict__ w, uint32_t c, float t,
                                              float (&res)[DIM]) {
    const double td = static_cast<double>(t);
    const T *__restrict__ Wp = w + static_cast<size_t>(c) * (D + 1);
    const T *__restrict__ P = ctrl + static_cast<size_t>(c) * DIM * (D + 1);
    [[maybe_unused]] T wv[D + 1], row[D + 1] = {};
    if constexpr (AHEAD)
#pragma unroll
        for (int i = 0; i <= D; ++i) wv[i] = Wp[i];
    double W = 0.0;
#pragma unroll 1
    for (int k = 0; k <= DIM; ++k) {  // the weight, then the coordinates
        const T *__restrict__ Pk = P + (k > 0 ? k - 1 : 0) * (D + 1);
        double H[D + 1];
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            const double wi = static_cast<double>(to_f32<T>(AHEAD ? wv[i] : Wp[i]));
            H[i] = k > 0 ? wi * static_cast<double>(to_f32<T>(AHEAD ? row[i] : Pk[i])) : wi;
        }
        if constexpr (AHEAD) {
            const T *__restrict__ next = P + (k < DIM ? k : DIM - 1) * (D + 1);
#pragma unroll
            for (int i = 0; i <= D; ++i) row[i] = next[i];
        }
#pragma unroll
        for (int lvl = 1; lvl <= D; ++lvl)
#pragma unroll
            for (int i = 0; i <= D - lvl; ++i) H[i] = lerp(H[i], H[i + 1], td);
        if (k == 0) W = H[0];
#pragma unroll
        for (int e = 0; e < DIM; ++e) res[e] = k == e + 1 ? static_cast<float>(H[0] / W) : res[e];
    }
}

// r[k] / W of all coordinates, correctly rounded: one reciprocal for all of
// them, refined once, and per coordinate a quotient with one residual
// correction (4 instructions against 11 of a division of its own).  Valid
// while no step under- or overflows; otherwise the plain divisions.
template <int DIM, int CH>
__device__ __forceinline__ void divide_all(const float (&r)[CH], float W, float (&res)[DIM]) {
    constexpr uint32_t kLo = (127u - 40u) << 23, kHi = (127u + 40u) << 23;  // 2^-40, 2^40
    float big = 0.0f;
    uint32_t small = 0xffffffffu;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const uint32_t u = __float_as_uint(__builtin_fabsf(r[k]));
        big = __builtin_fmaxf(big, __builtin_fabsf(r[k]));
        small = min(small, u - 1u);  // zero passes
    }
    const uint32_t uw = __float_as_uint(__builtin_fabsf(W));
    const bool plain = !(uw >= kLo && uw <= kHi && __float_as_uint(big) <= kHi && small >= kLo);
    bool nan = false;  // (fmax drops a NaN)
#pragma unroll
    for (int k = 0; k < DIM; ++k) nan = nan || r[k] != r[k];
    if (plain || nan) {
#pragma unroll
        for (int k = 0; k < DIM; ++k) res[k] = r[k] / W;
        return;
    }
    float y = __builtin_amdgcn_rcpf(W);
    y = __builtin_fmaf(__builtin_fmaf(-W, y, 1.0f), y, y);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const float q = r[k] * y;
        res[k] = __builtin_copysignf(__builtin_fmaf(__builtin_fmaf(-W, q, r[k]), y, q), q);
    }
}

struct CurveArgs {
    const void *ctrl;      // storage of curves [c0, c0+n)
    const void *w;         // weights (rational) or nullptr
    const float *t;        // base of the full parameter array
    float *out;            // base of the full output array
    int64_t plane;         // total queries of the call (output plane stride)
    int64_t q0;            // first query of this launch (global index)
    int64_t c0;            // first curve of this launch
    uint32_t nq;           // queries in this launch
    FastDiv div_nt;        // division by n_t
    int per_object;        // t[n][n_t] vs t[n_t]
    float kappa;           // rational conditioning threshold (<= 0: off)
    uint32_t *n_fixed;     // nullable device counter
    bool t_in_out;         // the points overwrite the parameters (t a plane of out, say)
    // k_curves_mixed: queries per workgroup, curves it may touch, and whether the
    // planes lie alike to the 64-byte lines
    int chunk, slots, same;
};

// UNI: n_t is a multiple of 64, so each wavefront evaluates one curve; its
// index is made wave-uniform and the control points come in through scalar
// loads instead of 64 identical vector loads.
template <int D, int DIM, int F, bool RAT, typename T, bool UNI>
__global__ __launch_bounds__(kBlock) void k_curves(CurveArgs a) {
    const uint32_t ql = blockIdx.x * kBlock + threadIdx.x;
    if (ql >= a.nq) return;
    uint32_t cl = fdiv(ql, a.div_nt);
    if constexpr (UNI) cl = __builtin_amdgcn_readfirstlane(cl);
    const uint32_t j = ql - cl * a.div_nt.d;
    const int64_t qg = a.q0 + ql;
    const float t = a.per_object ? a.t[qg] : a.t[j];

    constexpr int CH = DIM + (RAT ? 1 : 0);
    const T *__restrict__ P = static_cast<const T *>(a.ctrl) + static_cast<size_t>(cl) * DIM * (D + 1);
    float b[CH][D + 1];
#pragma unroll
    for (int k = 0; k < DIM; ++k)
#pragma unroll
        for (int i = 0; i <= D; ++i) b[k][i] = to_f32<T>(P[k * (D + 1) + i]);

    float r[CH];
    if constexpr (!RAT) {
        eval_channels<D, CH, F>(b, t, r);
#pragma unroll
        for (int k = 0; k < DIM; ++k) st_stream(a.out + k * a.plane + qg, r[k]);
    } else {
        const T *__restrict__ Wp = static_cast<const T *>(a.w) + static_cast<size_t>(cl) * (D + 1);
        bool allpos = true;
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            const float wi = to_f32<T>(Wp[i]);
            allpos = allpos && (wi > 0.0f);
            b[DIM][i] = wi;
#pragma unroll
            for (int k = 0; k < DIM; ++k) b[k][i] *= wi;
        }
        eval_channels<D, CH, F>(b, t, r);
        const float W = r[DIM];
        bool fix = false;
        if (a.kappa > 0.0f && !(allpos && W > 0.0f && W < __builtin_inff())) {
            float aw[1][D + 1];
#pragma unroll
            for (int i = 0; i <= D; ++i) aw[0][i] = __builtin_fabsf(b[DIM][i]);
            float A[1];
            eval_channels<D, 1, F>(aw, t, A);
            fix = (t == t) && !(A[0] <= a.kappa * __builtin_fabsf(W));
        }
        float res[DIM];
        if (fix) {
            rational_fp64<D, DIM, true, T>(static_cast<const T *>(a.ctrl), static_cast<const T *>(a.w), cl, t, res);
        } else {
            divide_all<DIM>(r, W, res);
        }
        if (a.n_fixed) {
            const uint64_t m = __ballot(fix);
            if (m != 0 && __lane_id() == static_cast<unsigned>(__ffsll(static_cast<long long>(m)) - 1))
                atomicAdd(a.n_fixed, static_cast<uint32_t>(__popcll(m)));
        }
#pragma unroll
        for (int k = 0; k < DIM; ++k) st_stream(a.out + k * a.plane + qg, res[k]);
    }
}

// A workgroup takes `chunk` consecutive queries, stages the control points of
// the curves they lie on in LDS -- widened, times their weights, or as Seiler
// terms, once per curve instead of once per query -- and evaluates up to four
// queries per thread from there.  Loading a curve per query took a vector load
// and a conversion per coefficient.
// The stores bypass the caches and want whole lines, so a chunk begins on one;
// where the coordinate planes don't lie alike (their distance is no multiple of
// 64 bytes) each plane takes its own part of the chunk, up to 31 queries apart,
// by way of LDS.
template <int D, int DIM, bool RAT>
struct MixedGeom {
    static constexpr int CH = DIM + (RAT ? 1 : 0);
    static constexpr int PAD = (D + 4) / 4 * 4;     // floats per row: whole 16-byte vectors
    static constexpr int CURVE = CH * PAD + 4;      // per curve; the last four: all weights positive
};

// Floats of a query's store past the last 128-byte line.
__device__ __forceinline__ uint32_t line_offset(const float *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p) >> 2) & 31u;
}

template <int D, int DIM, int F, bool RAT, typename T>
__global__ __launch_bounds__(kBlock) void k_curves_mixed(CurveArgs a) {
    using G = MixedGeom<D, DIM, RAT>;
    constexpr int CH = G::CH, PAD = G::PAD;
    extern __shared__ __align__(16) float lds[];
    float *__restrict__ out = a.out + a.q0;
    const uint32_t at = blockIdx.x * a.chunk;
    const uint32_t sh = a.same ? line_offset(out) : 31u;
    const uint32_t first = at > sh ? at - sh : 0;
    const uint32_t end = min(a.nq, at + a.chunk - (a.same ? sh : 0u));
    const int n = static_cast<int>(end - first);
    if (n <= 0) return;
    const uint32_t c_lo = fdiv(first, a.div_nt), s0 = first - c_lo * a.div_nt.d;
    const int n_c = static_cast<int>(fdiv(s0 + n - 1, a.div_nt)) + 1;
    const float *__restrict__ tq = a.per_object ? a.t + a.q0 + first : a.t;
    // parameter of query first + p (of the last one beyond), and its curve
    auto param = [&](int p, uint32_t &k) {
        const uint32_t q = min(p, n - 1);
        k = fdiv(s0 + q, a.div_nt);
        return tq[a.per_object ? q : s0 + q - k * a.div_nt.d];
    };
    uint32_t k_next;
    float t_next = param(threadIdx.x, k_next);  // on its way while the curves are staged
    const T *__restrict__ P = static_cast<const T *>(a.ctrl) + static_cast<size_t>(c_lo) * DIM * (D + 1);
    const T *__restrict__ Wp = RAT ? static_cast<const T *>(a.w) + static_cast<size_t>(c_lo) * (D + 1) : nullptr;
#pragma unroll 4
    for (int e = threadIdx.x; e < n_c * DIM * (D + 1); e += kBlock) {
        const int r = e / (D + 1), i = e - r * (D + 1);
        const int k = r / DIM, ch = r - k * DIM;
        float v = to_f32<T>(P[e]);
        if constexpr (RAT && F != FORM_SEILER) v *= to_f32<T>(Wp[k * (D + 1) + i]);
        lds[k * G::CURVE + ch * PAD + i] = v;
    }
    if constexpr (RAT) {
#pragma unroll 2
        for (int e = threadIdx.x; e < n_c * (D + 1); e += kBlock) {
            const int k = e / (D + 1), i = e - k * (D + 1);
            lds[k * G::CURVE + DIM * PAD + i] = to_f32<T>(Wp[e]);
        }
        for (int k = kBlock - 1 - threadIdx.x; k < n_c; k += kBlock) {
            bool allpos = true;
#pragma unroll
            for (int i = 0; i <= D; ++i) allpos = allpos && (to_f32<T>(Wp[k * (D + 1) + i]) > 0.0f);
            lds[k * G::CURVE + CH * PAD] = allpos ? 1.0f : 0.0f;
        }
    }
    __syncthreads();
    if constexpr (F == FORM_SEILER) {
        // rows to terms, in place; the weights, which the coordinates' rows need, last
        auto terms = [&](int first_ch, int n_ch) {
            for (int r = threadIdx.x; r < n_c * n_ch; r += kBlock) {
                const int k = r / n_ch, ch = first_ch + r - k * n_ch;
                float *curve = lds + k * G::CURVE, *row = curve + ch * PAD;
                float b[D + 1], sc[D + 1];
#pragma unroll
                for (int i = 0; i <= D; ++i) b[i] = row[i];
                if (RAT && ch < DIM) {
                    float w[D + 1];
#pragma unroll
                    for (int i = 0; i <= D; ++i) w[i] = curve[DIM * PAD + i];
                    seiler_terms_of_products<D>(b, w, sc);
                } else {
                    seiler_terms<D, float>(b, sc);
                }
#pragma unroll
                for (int i = 0; i <= D; ++i) row[i] = sc[i];
            }
            __syncthreads();
        };
        terms(0, DIM);
        if constexpr (RAT) terms(DIM, 1);
    }
    constexpr int FE = F == FORM_SEILER ? FORM_SEILER_PRE : F;  // from the staged data
    float *__restrict__ buf = lds + a.slots * G::CURVE;         // [DIM][chunk + 32] unless the planes lie alike
    const int pitch = a.chunk + 32;
    auto points = [&](auto same) {
#pragma unroll 1
        for (int p = threadIdx.x; p < n; p += kBlock) {
            const float t = t_next;
            const uint32_t kq = k_next;
            t_next = param(p + kBlock, k_next);
            const float *__restrict__ row = lds + kq * G::CURVE;
            float b[CH][D + 1], r[CH], res[DIM];
#pragma unroll
            for (int k = 0; k < CH; ++k)
#pragma unroll
                for (int e = 0; e <= D; ++e) b[k][e] = row[k * PAD + e];
            eval_channels<D, CH, FE>(b, t, r);
            if constexpr (!RAT) {
#pragma unroll
                for (int k = 0; k < DIM; ++k) res[k] = r[k];
            } else {
                const float W = r[DIM];
                const uint32_t cl = c_lo + kq;
                bool fix = false;
                if (a.kappa > 0.0f && !(row[CH * PAD] != 0.0f && W > 0.0f && W < __builtin_inff())) {
                    float aw[1][D + 1], A[1];
#pragma unroll
                    for (int e = 0; e <= D; ++e)
                        aw[0][e] = __builtin_fabsf(to_f32<T>(static_cast<const T *>(a.w)[static_cast<size_t>(cl) * (D + 1) + e]));
                    eval_channels<D, 1, F>(aw, t, A);
                    fix = (t == t) && !(A[0] <= a.kappa * __builtin_fabsf(W));
                }
                if (fix) rational_fp64<D, DIM, false, T>(static_cast<const T *>(a.ctrl), static_cast<const T *>(a.w), cl, t, res);
                else divide_all<DIM>(r, W, res);
                if (a.n_fixed) {
                    // (queries before `at` are the previous workgroup's to count)
                    const uint64_t m = __ballot(fix && (decltype(same)::value || first + p >= at));
                    if (m != 0 && __lane_id() == static_cast<unsigned>(__ffsll(static_cast<long long>(m)) - 1))
                        atomicAdd(a.n_fixed, static_cast<uint32_t>(__popcll(m)));
                }
            }
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                if constexpr (decltype(same)::value) st_stream(at_lane(out + k * a.plane + first, p), res[k]);
                else buf[k * pitch + p] = res[k];
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
    for (int k = 0; k < DIM; ++k) {
        float *__restrict__ oc = out + k * a.plane;
        const uint32_t sc = line_offset(oc), lo = at > sc ? 0 : sc - at;  // plane queries [at - sc + lo, ...)
        // (none in the last workgroup where the plane's end lies before its part)
        const uint32_t n_own = a.nq + sc > at ? min(static_cast<uint32_t>(a.chunk), a.nq + sc - at) : 0;
        float *__restrict__ to = oc + at - sc;
        const float *__restrict__ from = buf + k * pitch + static_cast<int>(at - sc - first);
        for (uint32_t p = threadIdx.x; p < n_own; p += kBlock)
            if (p >= lo) st_stream(at_lane(to, p), from[p]);
    }
}

// Seiler terms per (curve, coordinate): one thread per pair.
template <int D, typename T>
__global__ __launch_bounds__(kBlock) void k_to_seiler(const T *__restrict__ ctrl, float *__restrict__ seiler, uint32_t n_rows) {
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= n_rows) return;
    float b[D + 1], sc[D + 1];
#pragma unroll
    for (int i = 0; i <= D; ++i) b[i] = to_f32<T>(ctrl[static_cast<size_t>(r) * (D + 1) + i]);
    seiler_terms<D>(b, sc);
#pragma unroll
    for (int i = 0; i <= D; ++i) seiler[static_cast<size_t>(r) * (D + 1) + i] = sc[i];
}

// ---------------------------------------------------------------- host
// Which kernel.  Integral points of curves with n_t a multiple of 64 come from
// scalar-loaded control points (staging them in LDS: 10.0 against 9.7 us for
// 16384 cubics x 256), except in Seiler form of degree 5 and up, whose terms are
// then formed once per curve (65536 curves x 256, staged against scalar loads:
// degree 3 37.5 and 29.6 us, 4 38.1 and 34.4, 5 37.3 and 42.0, 7 33.3 and 60.5).
// Parameters that the points overwrite are read by one thread per query: a thread
// then reads no parameter but its own query's, where a staged workgroup evaluates
// up to 31 of the one before.
// Otherwise one thread per query is the faster in small calls, whose time is the
// chain of a workgroup's stages, and staging in large ones, whose time is the
// loads and conversions of a curve's coefficients for each of its queries.  The
// line lies the lower, the more staging saves: terms formed once (Seiler), high
// degrees, and curves of 64, 128, ... queries, few of them per workgroup; and
// higher for curves of under 12 queries, many of them per workgroup.  Queries
// from which on calls are staged, as log2, by degree (up to 5, 10, 15), from
// 7,000 random calls on rotating buffers: so chosen they take 1.1 % more time
// than with the better kernel each, all staged 16 % more, all with one thread per
// query 7 % (118 rational curves of degree 5 in 3D, BF16, x 45: 2.3 us with a
// thread per query, 3.3 staged; 9754 of degree 15 in 4D, FP16, Seiler form x 36:
// 10.7 and 5.6; 100,003 rational quintics x 50: 21.9 and 21.5).
// Curves of fewer than kMixedMinT queries are never staged (3,000,000 cubics x 1:
// 30 us with a thread per query, 36 staged).
constexpr uint32_t kMixedMinT = 8;

template <int F, bool RAT, int D>
constexpr int staged_log2() {
    constexpr int g = D <= 5 ? 0 : D <= 10 ? 1 : 2;
    constexpr int dc[2][3] = {{23, 23, 22}, {23, 22, 21}}, bern[2][3] = {{21, 20, 20}, {23, 22, 22}};
    constexpr int seiler[2][3] = {{21, 19, 17}, {22, 19, 18}}, terms[3] = {21, 20, 18};
    return F == FORM_DC ? dc[RAT][g] : F == FORM_BERN ? bern[RAT][g] : F == FORM_SEILER ? seiler[RAT][g] : terms[g];
}

template <int F, bool RAT, typename T, int D, int DIM>
void launch_curves_dd(CurveArgs a, hipStream_t s) {
    const uint32_t n_t = a.div_nt.d, flat = (a.nq + kBlock - 1) / kBlock;
    if constexpr (!RAT && (F != FORM_SEILER || D <= 4)) {
        if (n_t % 64 == 0) {
            hipLaunchKernelGGL((k_curves<D, DIM, F, RAT, T, true>), dim3(flat), dim3(kBlock), 0, s, a);
            return;
        }
    }
    const int from = staged_log2<F, RAT, D>() + (n_t < 12 ? 2 : 0) -
                     (n_t % 64 == 0 ? (F == FORM_SEILER ? 1 : 2) : RAT && F == FORM_BERN && n_t >= 40 ? 1 : 0);
    if (n_t < kMixedMinT || a.t_in_out || a.nq < 1u << from) {
        hipLaunchKernelGGL((k_curves<D, DIM, F, RAT, T, false>), dim3(flat), dim3(kBlock), 0, s, a);
        return;
    }
    // chunks of 1024 queries, fewer in calls too small to give every CU two
    // workgroups and where the curves of so many would not leave a CU four
    using G = MixedGeom<D, DIM, RAT>;
    a.same = DIM == 1 || a.plane % 16 == 0;
    size_t floats = 0;
    for (int want = a.nq >= 1024u * 512 ? 1024 : a.nq >= 512u * 512 ? 512 : 256;; want /= 2) {
        a.chunk = a.same ? want : want - 32;  // with the planes' own first queries: whole threads
        const uint32_t span = a.chunk + (a.same ? 0 : 31);
        a.slots = static_cast<int>((span + n_t - 2) / n_t + 1);
        floats = static_cast<size_t>(a.slots) * G::CURVE + (a.same ? 0 : DIM * (a.chunk + 32));
        if (floats <= 10240 || want == 128) break;
    }
    const uint32_t blocks = static_cast<uint32_t>((static_cast<uint64_t>(a.nq) + 31 + a.chunk - 1) / a.chunk);
    hipLaunchKernelGGL((k_curves_mixed<D, DIM, F, RAT, T>), dim3(blocks), dim3(kBlock), floats * sizeof(float), s, a);
}

template <int F, bool RAT, typename T, int D>
int launch_curves_d(int dim, const CurveArgs &a, hipStream_t s) {
    switch (dim) {
        case 1: launch_curves_dd<F, RAT, T, D, 1>(a, s); break;
        case 2: launch_curves_dd<F, RAT, T, D, 2>(a, s); break;
        case 3: launch_curves_dd<F, RAT, T, D, 3>(a, s); break;
        case 4: launch_curves_dd<F, RAT, T, D, 4>(a, s); break;
        default: return fail(BZ_ERR_SHAPE, "dim %d out of range", dim);
    }
    BZ_CHECK_LAUNCH("k_curves");
    return BZ_OK;
}

// Launch one chunk of curve queries for form F (rational when RAT) with
// control points stored as T; explicitly instantiated per form in its own
// translation unit so the 15 x 4 specialisations compile in parallel.
template <int F, bool RAT, typename T>
int launch_curves_t(int degree, int dim, const CurveArgs &a, hipStream_t s) {
    switch (degree) {
        case 1: return launch_curves_d<F, RAT, T, 1>(dim, a, s);
        case 2: return launch_curves_d<F, RAT, T, 2>(dim, a, s);
        case 3: return launch_curves_d<F, RAT, T, 3>(dim, a, s);
        case 4: return launch_curves_d<F, RAT, T, 4>(dim, a, s);
        case 5: return launch_curves_d<F, RAT, T, 5>(dim, a, s);
        case 6: return launch_curves_d<F, RAT, T, 6>(dim, a, s);
        case 7: return launch_curves_d<F, RAT, T, 7>(dim, a, s);
        case 8: return launch_curves_d<F, RAT, T, 8>(dim, a, s);
        case 9: return launch_curves_d<F, RAT, T, 9>(dim, a, s);
        case 10: return launch_curves_d<F, RAT, T, 10>(dim, a, s);
        case 11: return launch_curves_d<F, RAT, T, 11>(dim, a, s);
        case 12: return launch_curves_d<F, RAT, T, 12>(dim, a, s);
        case 13: return launch_curves_d<F, RAT, T, 13>(dim, a, s);
        case 14: return launch_curves_d<F, RAT, T, 14>(dim, a, s);
        case 15: return launch_curves_d<F, RAT, T, 15>(dim, a, s);
        default: return fail(BZ_ERR_SHAPE, "degree %d out of range", degree);
    }
}

}  // namespace bzi
