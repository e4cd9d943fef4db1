// Adjoint of curve evaluation and a fused least-squares fitting step (loss,
// gradients through the hodograph, Adam) for gfx950.
//
// One wavefront per curve: the 64 lanes walk the curve's n_t parameters, each
// lane accumulating its share of dL/db (and dL/dw) in registers; a butterfly
// of cross-lane shuffles then sums the partials, so the per-curve reduction is
// deterministic and needs no atomics.  dL/dt is per query and is written by
// the lane that owns the query.
#include <cmath>

#include "fit_impl.h"

namespace bzi {

extern template int launch_fit_run_d<1>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<2>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<3>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<4>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<5>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<6>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<7>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<8>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<9>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<10>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<11>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<12>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<13>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<14>(int, const FitArgs &, const FitBias &, int, hipStream_t);
extern template int launch_fit_run_d<15>(int, const FitArgs &, const FitBias &, int, hipStream_t);

namespace {

struct AdjArgs {
    const float *ctrl;
    const float *w;
    const float *t;
    const float *gout;
    float *gctrl;
    float *gw;
    float *gt;
    int64_t n_curves;
    int64_t n_t;
    int64_t plane;
    int per_object;
};

template <int D, int DIM, bool RAT>
__global__ __launch_bounds__(kBlock) void k_adjoint(AdjArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t c = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6));
    if (c >= a.n_curves) return;
    float b[DIM][D + 1], wv[D + 1];
#pragma unroll
    for (int k = 0; k < DIM; ++k)
#pragma unroll
        for (int i = 0; i <= D; ++i) b[k][i] = a.ctrl[(c * DIM + k) * (D + 1) + i];
#pragma unroll
    for (int i = 0; i <= D; ++i) wv[i] = RAT ? a.w[c * (D + 1) + i] : 1.0f;
    float gb[DIM][D + 1] = {}, gwv[D + 1] = {};
    for (int64_t j = lane; j < a.n_t; j += 64) {
        const int64_t q = c * a.n_t + j;
        const float t = a.per_object ? a.t[q] : a.t[j];
        float B[D + 1], W, C[DIM], dC[DIM], g[DIM];
        curve_and_derivative<D, DIM, RAT>(b, wv, t, B, W, C, dC);
        float dt = 0.0f;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            g[k] = a.gout[k * a.plane + q];
            dt = __builtin_fmaf(g[k], dC[k], dt);
        }
        if (a.gt) a.gt[q] = dt;
        const float iW = RAT ? 1.0f / W : 1.0f;
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            const float s = RAT ? wv[i] * B[i] * iW : B[i];
#pragma unroll
            for (int k = 0; k < DIM; ++k) gb[k][i] = __builtin_fmaf(g[k], s, gb[k][i]);
            if constexpr (RAT) {
                float acc = 0.0f;
#pragma unroll
                for (int k = 0; k < DIM; ++k) acc = __builtin_fmaf(g[k], b[k][i] - C[k], acc);
                gwv[i] = __builtin_fmaf(B[i] * iW, acc, gwv[i]);
            }
        }
    }
    if (a.gctrl) {
#pragma unroll
        for (int k = 0; k < DIM; ++k)
#pragma unroll
            for (int i = 0; i <= D; ++i) {
                const float v = wave_sum(gb[k][i]);
                if (lane == 0) a.gctrl[(c * DIM + k) * (D + 1) + i] = v;
            }
    }
    if (RAT && a.gw) {
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            const float v = wave_sum(gwv[i]);
            if (lane == 0) a.gw[c * (D + 1) + i] = v;
        }
    }
}

// Fused step: L = (1/M) sum |C(t) - y|^2, gradients, Adam on t (clamped to
// [0,1]) and on the control points.  All gradients use the parameters as they
// were at the start of the step.  Two curves per wavefront: lanes 0-31 work
// on curve 2w, lanes 32-63 on curve 2w+1, so one DPP butterfly reduces the
// per-curve sums of both.
template <int D, int DIM>
__global__ __launch_bounds__(kBlock) void k_fit_step(FitArgs a) {
    constexpr int NP = DIM * (D + 1);
    constexpr int CPW = NP <= 32 ? 2 : 1;  // curves per wavefront
    constexpr int L = 64 / CPW;            // lanes per curve
    const int lane = threadIdx.x & 63, sub = lane % L;
    const int64_t c0 = CPW * static_cast<int64_t>(__builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)));
    if (c0 >= a.n_curves) return;
    const bool has1 = CPW == 2 && c0 + 1 < a.n_curves;
    const int64_t c = (lane < L || !has1) ? c0 : c0 + 1;
    const bool live = lane < L || has1;  // the upper half idles when the curve count is odd
    // both curves' control points are wave-uniform: scalar loads, then a select
    float b[DIM][D + 1], wv[D + 1] = {};
#pragma unroll
    for (int k = 0; k < DIM; ++k)
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            const float v0 = a.ctrl[c0 * NP + k * (D + 1) + i];
            const float v1 = a.ctrl[(has1 ? c0 + 1 : c0) * NP + k * (D + 1) + i];
            b[k][i] = lane < L ? v0 : v1;
        }
    const int64_t pidx = c * NP + (sub < NP ? sub : 0);
    const float p_own = a.ctrl[pidx];
    float m_own = a.m_c[pidx], v_own = a.v_c[pidx];
    float mine = 0.0f, loss_sum = 0.0f;
    // blocks of kFitSpl samples per lane (see there)
    for (int64_t j0 = 0; j0 == 0 || j0 < a.n_t; j0 += kFitSpl * L) {
        const int64_t j1 = min(a.n_t, j0 + kFitSpl * L);
        float gb[DIM][D + 1] = {};
        float loss = 0.0f;
        for (int64_t j = j0 + sub; live && j < j1; j += L) {
            const int64_t q = c * a.n_t + j;
            const float t = a.t[q];
            float mt = a.m_t[q], vt = a.v_t[q];
            float yv[DIM];
#pragma unroll
            for (int k = 0; k < DIM; ++k) yv[k] = a.y[k * a.plane + q];
            float B[D + 1], W, C[DIM], dC[DIM];
            curve_and_derivative<D, DIM, false>(b, wv, t, B, W, C, dC);
            float dt = 0.0f;
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                const float r = C[k] - yv[k];
                loss = __builtin_fmaf(r, r, loss);
                const float g = 2.0f * r * a.inv_m;
                dt = __builtin_fmaf(g, dC[k], dt);
#pragma unroll
                for (int i = 0; i <= D; ++i) gb[k][i] = __builtin_fmaf(g, B[i], gb[k][i]);
            }
            float tn = adam(t, dt, &mt, &vt, a);
            tn = tn < 0.0f ? 0.0f : (tn > 1.0f ? 1.0f : tn);
            a.t[q] = tn;
            a.m_t[q] = mt;
            a.v_t[q] = vt;
        }
        loss = CPW == 2 ? half_sum(loss) : wave_sum(loss);
        const float blk = reduce_grads<D, DIM, CPW>(gb, sub);
        loss_sum = j0 == 0 ? loss : loss_sum + loss;
        mine = j0 == 0 ? blk : mine + blk;
    }
    if (a.loss_part && sub == 0 && live) a.loss_part[c] = loss_sum * a.inv_m;
    if (sub < NP && live) {
        const float pn = adam(p_own, mine, &m_own, &v_own, a);
        a.ctrl[pidx] = pn;
        a.m_c[pidx] = m_own;
        a.v_c[pidx] = v_own;
    }
}

// Gradient of the least-squares loss L = inv_m * sum |C(t) - y|^2 without an
// optimiser step: per-curve loss contributions, dL/db (one sum per control
// point, by the same reductions as the fused step) and dL/dt per query.  The
// lane mapping is that of k_fit_step (two curves per wavefront when a curve
// has at most 32 control-point coordinates); nothing is updated in place.
struct L2Args {
    const float *ctrl, *t, *y;
    float *loss_part, *gctrl, *gt;
    int64_t n_curves, n_t, plane;
    float inv_m;
};

template <int D, int DIM>
__global__ __launch_bounds__(kBlock) void k_l2_adjoint(L2Args a) {
    constexpr int NP = DIM * (D + 1);
    constexpr int CPW = NP <= 32 ? 2 : 1;
    constexpr int L = 64 / CPW;
    const int lane = threadIdx.x & 63, sub = lane % L;
    const int64_t c0 = CPW * static_cast<int64_t>(__builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)));
    if (c0 >= a.n_curves) return;
    const bool has1 = CPW == 2 && c0 + 1 < a.n_curves;
    const int64_t c = (lane < L || !has1) ? c0 : c0 + 1;
    const bool live = lane < L || has1;
    float b[DIM][D + 1], wv[D + 1] = {};
#pragma unroll
    for (int k = 0; k < DIM; ++k)
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            const float v0 = a.ctrl[c0 * NP + k * (D + 1) + i];
            const float v1 = a.ctrl[(has1 ? c0 + 1 : c0) * NP + k * (D + 1) + i];
            b[k][i] = lane < L ? v0 : v1;
        }
    float gb[DIM][D + 1] = {};
    float loss = 0.0f;
    for (int64_t j = sub; live && j < a.n_t; j += L) {
        const int64_t q = c * a.n_t + j;
        const float t = a.t[q];
        float yv[DIM];
#pragma unroll
        for (int k = 0; k < DIM; ++k) yv[k] = a.y[k * a.plane + q];
        float B[D + 1], W, C[DIM], dC[DIM];
        curve_and_derivative<D, DIM, false>(b, wv, t, B, W, C, dC);
        float dt = 0.0f;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            const float r = C[k] - yv[k];
            loss = __builtin_fmaf(r, r, loss);
            const float g = 2.0f * r * a.inv_m;
            dt = __builtin_fmaf(g, dC[k], dt);
#pragma unroll
            for (int i = 0; i <= D; ++i) gb[k][i] = __builtin_fmaf(g, B[i], gb[k][i]);
        }
        if (a.gt) a.gt[q] = dt;
    }
    if (a.loss_part) {
        loss = CPW == 2 ? half_sum(loss) : wave_sum(loss);
        if (sub == 0 && live) a.loss_part[c] = loss * a.inv_m;
    }
    if (a.gctrl) {
        const float mine = reduce_grads<D, DIM, CPW>(gb, sub);
        if (sub < NP && live) a.gctrl[c * NP + sub] = mine;
    }
}

int launch_fit_run(int degree, int dim, const FitArgs &a, const FitBias &bias, int n_steps, hipStream_t s) {
    switch (degree) {
        case 1: return launch_fit_run_d<1>(dim, a, bias, n_steps, s);
        case 2: return launch_fit_run_d<2>(dim, a, bias, n_steps, s);
        case 3: return launch_fit_run_d<3>(dim, a, bias, n_steps, s);
        case 4: return launch_fit_run_d<4>(dim, a, bias, n_steps, s);
        case 5: return launch_fit_run_d<5>(dim, a, bias, n_steps, s);
        case 6: return launch_fit_run_d<6>(dim, a, bias, n_steps, s);
        case 7: return launch_fit_run_d<7>(dim, a, bias, n_steps, s);
        case 8: return launch_fit_run_d<8>(dim, a, bias, n_steps, s);
        case 9: return launch_fit_run_d<9>(dim, a, bias, n_steps, s);
        case 10: return launch_fit_run_d<10>(dim, a, bias, n_steps, s);
        case 11: return launch_fit_run_d<11>(dim, a, bias, n_steps, s);
        case 12: return launch_fit_run_d<12>(dim, a, bias, n_steps, s);
        case 13: return launch_fit_run_d<13>(dim, a, bias, n_steps, s);
        case 14: return launch_fit_run_d<14>(dim, a, bias, n_steps, s);
        default: return launch_fit_run_d<15>(dim, a, bias, n_steps, s);
    }
}

template <int D, bool RAT>
int launch_adj_d(int dim, const AdjArgs &a, hipStream_t s, uint32_t blocks) {
    switch (dim) {
        case 1: hipLaunchKernelGGL((k_adjoint<D, 1, RAT>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_adjoint<D, 2, RAT>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_adjoint<D, 3, RAT>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_adjoint<D, 4, RAT>), dim3(blocks), dim3(kBlock), 0, s, a); break;
    }
    BZ_CHECK_LAUNCH("k_adjoint");
    return BZ_OK;
}

template <bool RAT>
int launch_adj(int degree, int dim, const AdjArgs &a, hipStream_t s, uint32_t blocks) {
    switch (degree) {
        case 1: return launch_adj_d<1, RAT>(dim, a, s, blocks);
        case 2: return launch_adj_d<2, RAT>(dim, a, s, blocks);
        case 3: return launch_adj_d<3, RAT>(dim, a, s, blocks);
        case 4: return launch_adj_d<4, RAT>(dim, a, s, blocks);
        case 5: return launch_adj_d<5, RAT>(dim, a, s, blocks);
        case 6: return launch_adj_d<6, RAT>(dim, a, s, blocks);
        case 7: return launch_adj_d<7, RAT>(dim, a, s, blocks);
        case 8: return launch_adj_d<8, RAT>(dim, a, s, blocks);
        case 9: return launch_adj_d<9, RAT>(dim, a, s, blocks);
        case 10: return launch_adj_d<10, RAT>(dim, a, s, blocks);
        case 11: return launch_adj_d<11, RAT>(dim, a, s, blocks);
        case 12: return launch_adj_d<12, RAT>(dim, a, s, blocks);
        case 13: return launch_adj_d<13, RAT>(dim, a, s, blocks);
        case 14: return launch_adj_d<14, RAT>(dim, a, s, blocks);
        default: return launch_adj_d<15, RAT>(dim, a, s, blocks);
    }
}

template <int D>
int launch_fit_d(int dim, const FitArgs &a, hipStream_t s) {
    const int cpw = dim * (D + 1) <= 32 ? 2 : 1;
    const uint32_t blocks = static_cast<uint32_t>((a.n_curves + 4 * cpw - 1) / (4 * cpw));
    switch (dim) {
        case 1: hipLaunchKernelGGL((k_fit_step<D, 1>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_fit_step<D, 2>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_fit_step<D, 3>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_fit_step<D, 4>), dim3(blocks), dim3(kBlock), 0, s, a); break;
    }
    BZ_CHECK_LAUNCH("k_fit_step");
    return BZ_OK;
}

int launch_fit(int degree, int dim, const FitArgs &a, hipStream_t s) {
    switch (degree) {
        case 1: return launch_fit_d<1>(dim, a, s);
        case 2: return launch_fit_d<2>(dim, a, s);
        case 3: return launch_fit_d<3>(dim, a, s);
        case 4: return launch_fit_d<4>(dim, a, s);
        case 5: return launch_fit_d<5>(dim, a, s);
        case 6: return launch_fit_d<6>(dim, a, s);
        case 7: return launch_fit_d<7>(dim, a, s);
        case 8: return launch_fit_d<8>(dim, a, s);
        case 9: return launch_fit_d<9>(dim, a, s);
        case 10: return launch_fit_d<10>(dim, a, s);
        case 11: return launch_fit_d<11>(dim, a, s);
        case 12: return launch_fit_d<12>(dim, a, s);
        case 13: return launch_fit_d<13>(dim, a, s);
        case 14: return launch_fit_d<14>(dim, a, s);
        default: return launch_fit_d<15>(dim, a, s);
    }
}

template <int D>
int launch_l2_d(int dim, const L2Args &a, hipStream_t s) {
    const int cpw = dim * (D + 1) <= 32 ? 2 : 1;
    const uint32_t blocks = static_cast<uint32_t>((a.n_curves + 4 * cpw - 1) / (4 * cpw));
    switch (dim) {
        case 1: hipLaunchKernelGGL((k_l2_adjoint<D, 1>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_l2_adjoint<D, 2>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_l2_adjoint<D, 3>), dim3(blocks), dim3(kBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_l2_adjoint<D, 4>), dim3(blocks), dim3(kBlock), 0, s, a); break;
    }
    BZ_CHECK_LAUNCH("k_l2_adjoint");
    return BZ_OK;
}

int launch_l2(int degree, int dim, const L2Args &a, hipStream_t s) {
    switch (degree) {
        case 1: return launch_l2_d<1>(dim, a, s);
        case 2: return launch_l2_d<2>(dim, a, s);
        case 3: return launch_l2_d<3>(dim, a, s);
        case 4: return launch_l2_d<4>(dim, a, s);
        case 5: return launch_l2_d<5>(dim, a, s);
        case 6: return launch_l2_d<6>(dim, a, s);
        case 7: return launch_l2_d<7>(dim, a, s);
        case 8: return launch_l2_d<8>(dim, a, s);
        case 9: return launch_l2_d<9>(dim, a, s);
        case 10: return launch_l2_d<10>(dim, a, s);
        case 11: return launch_l2_d<11>(dim, a, s);
        case 12: return launch_l2_d<12>(dim, a, s);
        case 13: return launch_l2_d<13>(dim, a, s);
        case 14: return launch_l2_d<14>(dim, a, s);
        default: return launch_l2_d<15>(dim, a, s);
    }
}

int check_fit(const char *fn, float *ctrl, float *t, const float *y, int64_t n_curves, int degree, int dim, int64_t n_t,
              float *m_ctrl, float *v_ctrl, float *m_t, float *v_t, float lr, float beta1, float beta2, float eps) {
    if (degree < 1 || degree > kMaxDegree || dim < 1 || dim > kMaxDim)
        return fail(BZ_ERR_SHAPE, "%s: degree %d / dim %d out of range", fn, degree, dim);
    if (n_curves < 0 || n_t < 0 || n_t > 1024) return fail(BZ_ERR_SHAPE, "%s: need 0 <= n_t <= 1024", fn);
    if (n_curves > (int64_t(1) << 31) - 1) return fail(BZ_ERR_SHAPE, "%s: too many curves", fn);
    if (!(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps >= 0.0f))
        return fail(BZ_ERR_SHAPE, "%s: bad Adam hyper-parameters", fn);
    if (n_curves == 0 || n_t == 0) return BZ_OK;
    if (!ctrl || !t || !y || !m_ctrl || !v_ctrl || !m_t || !v_t) return fail(BZ_ERR_NULL, "%s: missing array", fn);
    return BZ_OK;
}

FitArgs make_fit_args(float *ctrl, float *t, const float *y, int64_t n_curves, int64_t n_t, float *m_ctrl,
                      float *v_ctrl, float *m_t, float *v_t, int step, float lr, float beta1, float beta2, float eps,
                      float *loss_part) {
    FitArgs a;
    a.ctrl = ctrl;
    a.t = t;
    a.y = y;
    a.m_c = m_ctrl;
    a.v_c = v_ctrl;
    a.m_t = m_t;
    a.v_t = v_t;
    a.loss_part = loss_part;
    a.n_curves = n_curves;
    a.n_t = n_t;
    a.plane = n_curves * n_t;
    a.inv_m = static_cast<float>(1.0 / static_cast<double>(n_curves * n_t));
    a.lr = lr;
    a.b1 = beta1;
    a.b2 = beta2;
    a.eps = eps;
    a.ic1 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(beta1), step)));
    a.ic2 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(beta2), step)));
    return a;
}

}  // namespace
}  // namespace bzi

using namespace bzi;

extern "C" {

int bz_adjoint_bezier(const float *ctrl, const float *w, int64_t n_curves, int degree, int dim, const float *t,
                      int64_t n_t, int t_mode, const float *grad_out, float *grad_ctrl, float *grad_w, float *grad_t,
                      bz_stream stream) {
    return guarded("bz_adjoint_bezier", [&]() -> int {
        const char *fn = "bz_adjoint_bezier";
        if (degree < 1 || degree > kMaxDegree || dim < 1 || dim > kMaxDim)
            return fail(BZ_ERR_SHAPE, "%s: degree %d / dim %d out of range", fn, degree, dim);
        if (n_curves < 0 || n_t < 0) return fail(BZ_ERR_SHAPE, "%s: negative count", fn);
        if (t_mode != BZ_T_SHARED && t_mode != BZ_T_PER_OBJECT) return fail(BZ_ERR_SHAPE, "%s: bad t_mode", fn);
        if (grad_t && t_mode != BZ_T_PER_OBJECT) return fail(BZ_ERR_UNSUPPORTED, "%s: grad_t needs per-object t", fn);
        if (grad_w && !w) return fail(BZ_ERR_NULL, "%s: grad_w needs w", fn);
        if (n_curves > (int64_t(1) << 31) - 1) return fail(BZ_ERR_SHAPE, "%s: too many curves", fn);
        if (n_curves == 0 || n_t == 0) return BZ_OK;
        if (!ctrl || !t || !grad_out) return fail(BZ_ERR_NULL, "%s: ctrl, t and grad_out are required", fn);
        AdjArgs a{ctrl, w, t, grad_out, grad_ctrl, grad_w, grad_t, n_curves, n_t, n_curves * n_t,
                  t_mode == BZ_T_PER_OBJECT};
        const uint32_t blocks = static_cast<uint32_t>((n_curves + 3) / 4);
        const hipStream_t s = as_stream(stream);
        return w ? launch_adj<true>(degree, dim, a, s, blocks) : launch_adj<false>(degree, dim, a, s, blocks);
    });
}

int bz_l2_fit_adjoint(const float *ctrl, int64_t n_curves, int degree, int dim, const float *t, int64_t n_t,
                      const float *target, float *loss_part, float *grad_ctrl, float *grad_t, bz_stream stream) {
    return guarded("bz_l2_fit_adjoint", [&]() -> int {
        const char *fn = "bz_l2_fit_adjoint";
        if (degree < 1 || degree > kMaxDegree || dim < 1 || dim > kMaxDim)
            return fail(BZ_ERR_SHAPE, "%s: degree %d / dim %d out of range", fn, degree, dim);
        if (n_curves < 0 || n_t < 0) return fail(BZ_ERR_SHAPE, "%s: negative count", fn);
        if (n_curves > (int64_t(1) << 31) - 1) return fail(BZ_ERR_SHAPE, "%s: too many curves", fn);
        if (n_curves == 0 || n_t == 0) return BZ_OK;
        if (!ctrl || !t || !target) return fail(BZ_ERR_NULL, "%s: ctrl, t and target are required", fn);
        if (!aligned(ctrl, 4) || !aligned(t, 4) || !aligned(target, 4) || !aligned(loss_part, 4) ||
            !aligned(grad_ctrl, 4) || !aligned(grad_t, 4))
            return fail(BZ_ERR_ALIGN, "%s: FP32 arrays need 4-byte alignment", fn);
        L2Args a;
        a.ctrl = ctrl;
        a.t = t;
        a.y = target;
        a.loss_part = loss_part;
        a.gctrl = grad_ctrl;
        a.gt = grad_t;
        a.n_curves = n_curves;
        a.n_t = n_t;
        a.plane = n_curves * n_t;
        a.inv_m = static_cast<float>(1.0 / static_cast<double>(n_curves * n_t));
        return launch_l2(degree, dim, a, as_stream(stream));
    });
}

int bz_fit_adam_step(float *ctrl, float *t, const float *y, int64_t n_curves, int degree, int dim, int64_t n_t,
                     float *m_ctrl, float *v_ctrl, float *m_t, float *v_t, int step, float lr, float beta1, float beta2,
                     float eps, float *loss_part, bz_stream stream) {
    return guarded("bz_fit_adam_step", [&]() -> int {
        int rc = check_fit("bz_fit_adam_step", ctrl, t, y, n_curves, degree, dim, n_t, m_ctrl, v_ctrl, m_t, v_t, lr,
                           beta1, beta2, eps);
        if (rc || n_curves == 0 || n_t == 0) return rc;
        if (step < 1) return fail(BZ_ERR_SHAPE, "bz_fit_adam_step: step counts from 1");
        const FitArgs a = make_fit_args(ctrl, t, y, n_curves, n_t, m_ctrl, v_ctrl, m_t, v_t, step, lr, beta1, beta2,
                                        eps, loss_part);
        return launch_fit(degree, dim, a, as_stream(stream));
    });
}

int bz_fit_adam_run(float *ctrl, float *t, const float *y, int64_t n_curves, int degree, int dim, int64_t n_t,
                    float *m_ctrl, float *v_ctrl, float *m_t, float *v_t, int first_step, int n_steps, float lr,
                    float beta1, float beta2, float eps, float *loss_part, bz_stream stream) {
    return guarded("bz_fit_adam_run", [&]() -> int {
        const char *fn = "bz_fit_adam_run";
        int rc = check_fit(fn, ctrl, t, y, n_curves, degree, dim, n_t, m_ctrl, v_ctrl, m_t, v_t, lr, beta1, beta2, eps);
        if (rc || n_curves == 0 || n_t == 0 || n_steps == 0) return rc;
        if (first_step < 1 || n_steps < 0) return fail(BZ_ERR_SHAPE, "%s: steps count from 1", fn);
        const hipStream_t s = as_stream(stream);
        for (int i0 = 0; i0 < n_steps && rc == BZ_OK; i0 += kFitStepsPerLaunch) {
            const int n = std::min(kFitStepsPerLaunch, n_steps - i0);
            FitBias bias;
            for (int i = 0; i < n; ++i) {
                const FitArgs ai = make_fit_args(ctrl, t, y, n_curves, n_t, m_ctrl, v_ctrl, m_t, v_t, first_step + i0 + i,
                                                 lr, beta1, beta2, eps, loss_part);
                bias.v[i] = make_float2(ai.ic1, ai.ic2);
            }
            const FitArgs a = make_fit_args(ctrl, t, y, n_curves, n_t, m_ctrl, v_ctrl, m_t, v_t, first_step + i0, lr,
                                            beta1, beta2, eps, loss_part);
            rc = launch_fit_run(degree, dim, a, bias, n, s);
        }
        if (rc == BZ_OK) BZ_CHECK_HIP(hipStreamSynchronize(s));
        return rc;
    });
}

}  // extern "C"
