// Shared by the adjoint and the fitting kernels: per-curve reductions, the
// value and derivative of a curve, and the many-step fitting kernel, whose
// instantiations are spread over translation units by degree.
#pragma once
#include "curves_impl.h"

namespace bzi {

struct FitArgs {
    float *ctrl, *t;
    const float *y;
    float *m_c, *v_c, *m_t, *v_t;
    float *loss_part;
    int64_t n_curves, n_t, plane;
    float inv_m;        // 1 / (n_curves * n_t)
    float lr, b1, b2, eps;
    float ic1, ic2;  // 1 / (1 - b1^step), 1 / (1 - b2^step), rounded once from FP64
};

// Bias corrections (ic1, ic2) of the steps of one k_fit_run launch.
constexpr int kFitStepsPerLaunch = 128;
struct FitBias {
    float2 v[kFitStepsPerLaunch];
};

namespace {

// Sum over the 64 lanes: a DPP butterfly inside each 16-lane row (swap
// neighbours, swap pairs, mirror the 8-lane halves, mirror the row) leaves
// every lane holding its row's sum; the four row sums are then read lane by
// lane.  The result is wave-uniform.  No LDS traffic.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);  // row_half_mirror
    v += dpp_mov<0x140>(v);  // row_mirror
    const int b = __builtin_bit_cast(int, v);
    return (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)) +
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16))) +
           (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)) +
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48)));
}

// Sums over each 32-lane half of the wavefront (two curves per wave): the
// same row butterfly, then rows 0+1 and rows 2+3.  Lanes get their half's sum.
__device__ __forceinline__ float half_sum(float v) {
    v += dpp_mov<0xB1>(v);
    v += dpp_mov<0x4E>(v);
    v += dpp_mov<0x141>(v);
    v += dpp_mov<0x140>(v);
    const int b = __builtin_bit_cast(int, v);
    const float lo = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)) +
                     __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float hi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)) +
                     __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return (threadIdx.x & 32) ? hi : lo;
}

// Exchange with lane ^ D inside each 32-lane half: DPP for D = 1, 2 (quad
// permutations), ds_swizzle in xor mode (and-mask 31) for D = 4..16.
template <int D>
__device__ __forceinline__ float xor_lane(float v) {
    if constexpr (D == 1) return dpp_mov<0xB1>(v);
    else if constexpr (D == 2) return dpp_mov<0x4E>(v);
    else return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), (D << 10) | 0x1F));
}

// Reduce-scatter over a 32-lane half: NV values per lane in, and lane l of
// the half leaves with the half's sum of value l mod NV (NV = 16 or 32).  At
// each exchange a lane keeps the half of its values selected by one bit of
// its index (most significant first) and adds its partner's copy of that
// half, so the work halves with every exchange.
template <int NV, int D = NV / 2>
__device__ __forceinline__ void reduce_scatter_level(float (&v)[NV], int sub) {
    if constexpr (D >= 1) {
        const bool hi = (sub & D) != 0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float lo_v = v[j], hi_v = v[j + D];
            v[j] = (hi ? hi_v : lo_v) + xor_lane<D>(hi ? lo_v : hi_v);
        }
        reduce_scatter_level<NV, D / 2>(v, sub);
    }
}

template <int NV>
__device__ __forceinline__ float reduce_scatter32(float (&v)[NV], int sub) {
    reduce_scatter_level<NV>(v, sub);
    float r = v[0];
    if constexpr (NV == 16) r += xor_lane<16>(r);
    return r;
}

// Per-curve sums of the gradient partials gb[k][i], delivered to the lane
// that owns parameter sub = k*(D+1)+i (lanes past NP get unused values).
// Two curves per wavefront: reduce-scatter in each half; one curve: one
// wave sum per parameter.
template <int D, int DIM, int CPW>
__device__ __forceinline__ float reduce_grads(const float (&gb)[DIM][D + 1], int sub) {
    constexpr int NP = DIM * (D + 1);
    if constexpr (CPW == 2) {
        constexpr int NV = NP <= 16 ? 16 : 32;
        float v[NV];
#pragma unroll
        for (int e = 0; e < NV; ++e) v[e] = e < NP ? gb[e / (D + 1)][e % (D + 1)] : 0.0f;
        return reduce_scatter32<NV>(v, sub);
    } else {
        float mine = 0.0f;
#pragma unroll
        for (int k = 0; k < DIM; ++k)
#pragma unroll
            for (int i = 0; i <= D; ++i) {
                const float v = wave_sum(gb[k][i]);
                if (sub == k * (D + 1) + i) mine = v;
            }
        return mine;
    }
}

// Per query: value C, derivative C' (hodograph), and the basis B.
template <int D, int DIM, bool RAT>
__device__ __forceinline__ void curve_and_derivative(const float (&b)[DIM][D + 1], const float (&wv)[D + 1], float t,
                                                     float (&B)[D + 1], float &W, float (&C)[DIM], float (&dC)[DIM]) {
    bernstein_basis<D>(t, B);
    float Bm[D];
    bernstein_basis<D - 1>(t, Bm);
    if constexpr (!RAT) {
        W = 1.0f;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            C[k] = dot_basis<D>(B, b[k]);
            float d = 0.0f;
#pragma unroll
            for (int i = 0; i < D; ++i) d = __builtin_fmaf(b[k][i + 1] - b[k][i], Bm[i], d);
            dC[k] = static_cast<float>(D) * d;
        }
    } else {
        float wB[D + 1];
        W = 0.0f;
        float Wp = 0.0f;
#pragma unroll
        for (int i = 0; i <= D; ++i) {
            wB[i] = wv[i] * B[i];
            W += wB[i];
        }
#pragma unroll
        for (int i = 0; i < D; ++i) Wp = __builtin_fmaf(wv[i + 1] - wv[i], Bm[i], Wp);
        Wp *= static_cast<float>(D);
        const float iW = 1.0f / W;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            const float H = dot_basis<D>(wB, b[k]);
            float Hp = 0.0f;
#pragma unroll
            for (int i = 0; i < D; ++i) Hp = __builtin_fmaf(wv[i + 1] * b[k][i + 1] - wv[i] * b[k][i], Bm[i], Hp);
            Hp *= static_cast<float>(D);
            C[k] = H * iW;
            dC[k] = (Hp - C[k] * Wp) * iW;
        }
    }
}

// Adam update with the bias corrections as multiplications by host-side
// reciprocals and the hardware square root and reciprocal (v_sqrt_f32,
// v_rcp_f32, about 1 ulp) instead of correctly rounded division and square
// root sequences: the update is a heuristic step, and the IEEE sequences cost
// a third of the fitting step's instructions.  Every rounding step is written
// out so that all kernels produce identical bits.
__device__ __forceinline__ float adam_c(float p, float g, float *m, float *v, const FitArgs &a, float ic1, float ic2) {
    const float mm = __builtin_fmaf(a.b1, *m, (1.0f - a.b1) * g);
    const float vv = __builtin_fmaf(a.b2, *v, ((1.0f - a.b2) * g) * g);
    *m = mm;
    *v = vv;
    const float mh = mm * ic1, vh = vv * ic2;
    const float upd = mh * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(vh) + a.eps);
    return __builtin_fmaf(-a.lr, upd, p);
}

__device__ __forceinline__ float adam(float p, float g, float *m, float *v, const FitArgs &a) {
    return adam_c(p, g, m, v, a, a.ic1, a.ic2);
}

// The order in which a curve's gradient and loss are summed: blocks of
// kFitSpl samples per lane (a lane adds up its own in turn, the lanes are
// reduced), then the blocks in turn.  A block is what one wavefront of
// k_fit_run keeps in registers.
constexpr int kFitSpl = 8;

// Many fitting steps in one launch.  Curves are optimised independently, so
// wavefronts can keep their curves' samples, parameters and Adam moments in
// registers across all steps: HBM is read once and written once.  Each step
// performs exactly the arithmetic of k_fit_step, in the same order.  SPL:
// samples per lane; a curve of more than kFitSpl samples per lane takes
// `waves` wavefronts, one workgroup, which add up their sums through LDS (two
// buffers: one barrier per step) and all keep the curve's control points.
// Bound by the vector ALU: about 85 instructions per wavefront and sample of a
// cubic in 3D and 130 per step for the reduction and the update, so 8 samples
// per lane carry them better than 4.  16384 cubics of 200 samples: 6.9 us per
// step, 0.75 of the non-packed FP32 rate, against 22 us (and 230 us per call
// for building a graph) with a launch per step, which moves 36 bytes per sample.
// The bias corrections come in the kernel's arguments, so that a call needs no
// device memory.
template <int D, int DIM, int SPL>
__global__ __launch_bounds__(kBlock) void k_fit_run(FitArgs a, FitBias bias, int n_steps, int waves) {
    constexpr int NP = DIM * (D + 1);
    constexpr int CPW = NP <= 32 ? 2 : 1;
    constexpr int L = 64 / CPW;
    __shared__ float part[2][4][64];
    const int lane = threadIdx.x & 63, sub = lane % L;
    const int wv_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = waves == 1 ? 0 : wv_id;  // this wavefront's block of samples
    const int64_t pair = waves == 1 ? static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) + wv_id : blockIdx.x;
    const int64_t c0 = CPW * pair;
    if (c0 >= a.n_curves) return;
    const bool has1 = CPW == 2 && c0 + 1 < a.n_curves;
    const int64_t c = (lane < L || !has1) ? c0 : c0 + 1;
    const bool live = lane < L || has1;
    const int base = lane < L ? 0 : L;  // first lane of this lane's curve
    const int64_t pidx = c * NP + (sub < NP ? sub : 0);
    float p_own = a.ctrl[pidx], m_own = a.m_c[pidx], v_own = a.v_c[pidx];
    float ts[SPL], mts[SPL], vts[SPL], ys[SPL][DIM];
    const int j0 = sub + wave * kFitSpl * L;  // the lane's first sample; n_t <= 1024
    const int n_own = live ? static_cast<int>(a.n_t) - j0 : 0;  // sample s is the lane's own while s*L < n_own
    const int64_t q0 = c * a.n_t + j0;
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
        const int64_t q = s * L < n_own ? q0 + s * L : c * a.n_t;
        ts[s] = a.t[q];
        mts[s] = a.m_t[q];
        vts[s] = a.v_t[q];
#pragma unroll
        for (int k = 0; k < DIM; ++k) ys[s][k] = a.y[k * a.plane + q];
    }
    float b[DIM][D + 1], wv[D + 1] = {};
    float loss = 0.0f;
    const float two_inv_m = 2.0f * a.inv_m;
    for (int step = 0; step < n_steps; ++step) {
        // current control points of this lane's curve, from the owning lanes
        // (a lane-indexed permute through the LDS crossbar: one instruction per
        // parameter for both curves of the wave, none of them VALU)
        const int pb = __builtin_bit_cast(int, p_own);
#pragma unroll
        for (int k = 0; k < DIM; ++k)
#pragma unroll
            for (int i = 0; i <= D; ++i)
                b[k][i] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((base + k * (D + 1) + i) << 2, pb));
        const float2 bc = bias.v[step];
        float gb[DIM][D + 1] = {};
        loss = 0.0f;
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            if (s * L >= n_own) continue;
            float B[D + 1], W, C[DIM], dC[DIM];
            curve_and_derivative<D, DIM, false>(b, wv, ts[s], B, W, C, dC);
            float dt = 0.0f;
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                const float r = C[k] - ys[s][k];
                loss = __builtin_fmaf(r, r, loss);
                const float g = r * two_inv_m;  // = (2r) inv_m exactly: scaling by 2 commutes with rounding
                dt = __builtin_fmaf(g, dC[k], dt);
#pragma unroll
                for (int i = 0; i <= D; ++i) gb[k][i] = __builtin_fmaf(g, B[i], gb[k][i]);
            }
            float tn = adam_c(ts[s], dt, &mts[s], &vts[s], a, bc.x, bc.y);
            ts[s] = tn < 0.0f ? 0.0f : (tn > 1.0f ? 1.0f : tn);
        }
        float mine = reduce_grads<D, DIM, CPW>(gb, sub);
        if constexpr (SPL == kFitSpl) {
            if (waves > 1) {
                part[step & 1][wave][lane] = mine;
                __syncthreads();
                mine = part[step & 1][0][lane];
                for (int w = 1; w < waves; ++w) mine += part[step & 1][w][lane];
            }
        }
        if (sub < NP && live) p_own = adam_c(p_own, mine, &m_own, &v_own, a, bc.x, bc.y);
    }
    // only the last step's loss is reported, so only it is summed over the lanes
    loss = CPW == 2 ? half_sum(loss) : wave_sum(loss);
    if constexpr (SPL == kFitSpl) {
        if (waves > 1) {
            part[n_steps & 1][wave][lane] = loss;
            __syncthreads();
            loss = part[n_steps & 1][0][lane];
            for (int w = 1; w < waves; ++w) loss += part[n_steps & 1][w][lane];
        }
    }
    if (wave == 0) {
        if (a.loss_part && sub == 0 && live) a.loss_part[c] = loss * a.inv_m;
        if (sub < NP && live) {
            a.ctrl[pidx] = p_own;
            a.m_c[pidx] = m_own;
            a.v_c[pidx] = v_own;
        }
    }
#pragma unroll
    for (int s = 0; s < SPL; ++s)
        if (s * L < n_own) {
            const int64_t q = q0 + s * L;
            a.t[q] = ts[s];
            a.m_t[q] = mts[s];
            a.v_t[q] = vts[s];
        }
}

// Workgroups: a curve (pair) of several wavefronts is one workgroup; single
// wavefronts share one of four while they fill the chip, else have their own.
template <int D, int DIM>
int launch_fit_run_dd(const FitArgs &a, const FitBias &bias, int n_steps, hipStream_t s) {
    constexpr int NP = DIM * (D + 1);
    constexpr int L = NP <= 32 ? 32 : 64;
    const int64_t pairs = (a.n_curves * L + 63) / 64;
    const int spl = static_cast<int>((a.n_t + L - 1) / L);
    const int waves = (spl + kFitSpl - 1) / kFitSpl;  // n_t <= 1024: at most 4
    const int per = waves > 1 ? 1 : pairs >= 8192 ? 4 : 1;
    const dim3 blocks(static_cast<uint32_t>((pairs + per - 1) / per)), threads(64 * (waves > 1 ? waves : per));
    if (spl <= 1) hipLaunchKernelGGL((k_fit_run<D, DIM, 1>), blocks, threads, 0, s, a, bias, n_steps, 1);
    else if (spl <= 2) hipLaunchKernelGGL((k_fit_run<D, DIM, 2>), blocks, threads, 0, s, a, bias, n_steps, 1);
    else if (spl <= 4) hipLaunchKernelGGL((k_fit_run<D, DIM, 4>), blocks, threads, 0, s, a, bias, n_steps, 1);
    else hipLaunchKernelGGL((k_fit_run<D, DIM, kFitSpl>), blocks, threads, 0, s, a, bias, n_steps, waves);
    BZ_CHECK_LAUNCH("k_fit_run");
    return BZ_OK;
}

}  // namespace

template <int D>
int launch_fit_run_d(int dim, const FitArgs &a, const FitBias &bias, int n_steps, hipStream_t s) {
    switch (dim) {
        case 1: return launch_fit_run_dd<D, 1>(a, bias, n_steps, s);
        case 2: return launch_fit_run_dd<D, 2>(a, bias, n_steps, s);
        case 3: return launch_fit_run_dd<D, 3>(a, bias, n_steps, s);
        default: return launch_fit_run_dd<D, 4>(a, bias, n_steps, s);
    }
}

}  // namespace bzi
