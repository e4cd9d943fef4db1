// Mixed batches (integral / rational Bezier curves of degree 1..15 and cubic
// NURBS) evaluated by one persistent launch on gfx950.
//
// Plan (host, once): objects are sorted into uniform classes (kind, degree)
// so that every 256-query tile, and hence every wavefront, runs one code path;
// NURBS control points are gathered with their weights, beside their knots and
// a table for the per-query span lookup; tiles are ordered by estimated cost,
// heaviest first.
// Evaluation (batched_impl.h): a grid of (CUs x occupancy) workgroups takes
// tiles round-robin or from an atomic counter; the last workgroup to finish
// resets the counters, so consecutive launches (and graph replays) need no
// memset.  (The 16 lanes that evaluate one object load the same addresses,
// which the memory pipeline merges into one access; sharing the coefficients
// by DPP row broadcasts instead was measured slower.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <numeric>
#include <vector>

#include "batched_impl.h"

struct bz_plan_s;

namespace bzi {
namespace {

// Plan-time gather of control points (and weights of rational objects) into
// class-sorted, contiguous order: sorted object i of class c lands at
// ctrl_base(c) + slot*(d+1)*dim.  One thread per sorted object.
template <typename U>
__global__ __launch_bounds__(kBlock) void k_gather_sorted(int64_t n_sorted, const int32_t *__restrict__ perm,
                                                          const int64_t *__restrict__ cp_offset,
                                                          const ClassInfo *__restrict__ classes, int n_classes, int dim,
                                                          const U *__restrict__ ctrl, const U *__restrict__ w,
                                                          U *__restrict__ ctrl_s, U *__restrict__ w_s) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n_sorted) return;
    int c = 0;
    while (c + 1 < n_classes && classes[c + 1].first <= i) ++c;
    const ClassInfo ci = classes[c];
    if (ci.kind == 2) return;
    const int64_t slot = i - ci.first, o = perm[i];
    const int n = class_ncp(ci.kind, ci.degree) * dim;
    const U *src = ctrl + cp_offset[o] * dim;
    U *dst = ctrl_s + ci.ctrl_base + slot * n;
    for (int e = 0; e < n; ++e) dst[e] = src[e];
    if (ci.kind == 1 || ci.kind == 3)
        for (int e = 0; e <= ci.degree; ++e) w_s[ci.w_base + slot * (ci.degree + 1) + e] = w[cp_offset[o] + e];
}

// Plan-time weight check: flags[o] = 1 when a rational or NURBS object has a
// weight that is not positive (zero, negative or NaN).  One thread per object.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_weight_flags(int64_t n_obj, const uint16_t *__restrict__ kind_degree,
                                                         const int64_t *__restrict__ cp_offset, const T *__restrict__ w,
                                                         uint8_t *__restrict__ flags) {
    const int64_t o = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (o >= n_obj) return;
    uint8_t f = 0;
    const int kind = kind_degree[o] >> 8;
    if (kind == 1 || kind == 2)
        for (int64_t i = cp_offset[o]; i < cp_offset[o + 1]; ++i) f |= !(to_f32<T>(w[i]) > 0.0f);
    flags[o] = f;
}

// Plan-time copy of the NURBS control points, point by point with the weight
// last (storage bits unchanged).  One wavefront per NURBS.
template <typename U>
__global__ __launch_bounds__(kBlock) void k_gather_nurbs(int n_nurbs, const int64_t *__restrict__ nurbs_obj,
                                                         const int64_t *__restrict__ cp_offset,
                                                         const NurbsHead *__restrict__ head, int dim,
                                                         const U *__restrict__ ctrl, const U *__restrict__ w,
                                                         U *__restrict__ pts) {
    const int r = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (r >= n_nurbs) return;
    const int64_t cp = cp_offset[nurbs_obj[r]];
    const int64_t ncp = cp_offset[nurbs_obj[r] + 1] - cp;
    const int H = dim + 1;
    const U *P = ctrl + cp * dim;
    U *dst = pts + static_cast<int64_t>(head[r].cp0) * H;
    for (int64_t e = threadIdx.x & 63; e < ncp * H; e += 64) {
        const int64_t i = e / H, k = e - i * H;
        dst[e] = k == dim ? w[cp + i] : P[k * ncp + i];
    }
}

// Header and span table of one NURBS (see NurbsHead): for bucket m, the first
// span whose end lies in bucket m or later; a parameter of bucket m then lies in
// spans tab[m] .. tab[m+1], because the bucket function is monotone.  u: its
// ncp+4 knots; spans: the first knots of its non-empty spans.  Returns false if
// an entry is out of range (which the construction excludes; checked before
// anything reaches the device).
bool add_nurbs(const float *u, int64_t ncp, const std::vector<int32_t> &spans, int64_t cp0,
               std::vector<NurbsHead> &head, std::vector<uint16_t> &tab, std::vector<int> &bk) {
    NurbsHead h{};
    const int n = static_cast<int>(spans.size()), M = 2 * n;
    h.cp0 = static_cast<int32_t>(cp0);
    h.lo = u[kNurbsP];
    h.hi = u[ncp];
    h.inv_h = static_cast<float>(M) / (h.hi - h.lo);
    if (!std::isfinite(h.inv_h)) h.inv_h = 0.0f;  // one bucket holds every span
    if (ncp > 65535) {
        h.tab0 = -1;
        h.n_buckets = spans.back();
        head.push_back(h);
        return true;
    }
    h.tab0 = static_cast<int32_t>(tab.size());
    h.n_buckets = M;
    bk.resize(n);
    for (int i = 0; i < n; ++i) bk[i] = nurbs_bucket(u[spans[i] + 1], h.lo, h.inv_h, M);  // the span's end
    int i = 0;
    for (int m = 0; m <= M; ++m) {
        while (i < n - 1 && bk[i] < m) ++i;
        tab.push_back(static_cast<uint16_t>(spans[i]));
        if (spans[i] < kNurbsP || spans[i] >= ncp) return false;
    }
    head.push_back(h);
    return true;
}

// Tile layout of a plan that is not tuned: sub-tiles per tile, queries per lane,
// objects per window of the tile order (see build_tiles).
struct Layout {
    uint32_t qpt, vq, window;
};

// Of the layouts for the row length, the first that gives every CU a tile, for
// a tile's sub-tiles and a lane's queries run one after another: 32,000 objects
// x 16 (FP32) take 12.5 us with 168 tiles of 4 sub-tiles x 4 queries, 8.3 with
// 513 of 4 x 1; 87,000: 16.7 with 438 of 4 x 4, 17.8 with 1455 of 4 x 1; 6,500 x
// 8: 7.0 with 32 of 4 x 4, 5.6 with 219 of 1 x 1.
// Rows of n_t parameters or points that are whole 64-byte pieces are best read
// and written four at a time, in large windows (2^20 curves x 16: 138 us).
// Other rows share their pieces with their neighbours', which belong to other
// classes: smaller windows bring those together in the caches (400,000 objects
// x 10: 74 us with windows of 2^17, 66 with 2^14; 300,000 x 25: 94 and 83), one
// query per lane spreads short rows less (900,000 x 8 in windows of 2^15: 156 us
// with 4 x 4, 138 with 4 x 1; 400,000 x 12: 82 and 68), and of longer ones two
// sub-tiles do better than four (300,000 x 24: 64 us, 72 with four or with one
// query per lane).
// De Casteljau is quadratic in the degree, and rows of n_t % 16 == 0 take four
// queries per lane once the launch is long beside its heaviest tile: batches of up
// to degree 7 from two tiles of 4096 queries per CU on, 4 x 4; of up to 12 from
// four of 2048 on, 2 x 4, and 4 x 4 again from 16 of 4096; of up to 15 from twelve
// of 2048, 2 x 4 (FP32, curves and NURBS x 16 on rotating inputs: 262,144 of up to
// degree 5, 4 x 4 23.0 us, 2 x 4 25.9, 4 x 1 30.4; 262,144 of up to 12, 43, 42 and
// 42; 393,216 73, 65 and 77; 393,216 of up to 15, 90, 79 and 87; 16,384 of up to
// 15, 33, 19 and 13).  Other rows: 4 x 4 queries of degree 15 in turn are a long
// tail until every CU has 16 tiles of 2048 queries, and 2 x 4 suffice from there on.
Layout default_layout(const std::vector<ClassInfo> &cls, int method, int64_t n_t, uint32_t cus) {
    std::vector<Layout> choices;
    if (method == BZ_DECASTELJAU && n_t % 4 == 0 && n_t >= 16) {
        const uint32_t win = n_t % 16 == 0 ? 1u << 17 : 1u << 15;
        int64_t queries = 0;
        int degree = 1;
        for (const ClassInfo &ci : cls) {
            queries += ci.count * n_t;
            degree = std::max(degree, ci.kind == 4 ? 6 : ci.degree);  // (a bicubic patch: 3 + 3)
        }
        const int64_t per_cu = queries / cus;
        if (n_t % 16 == 0) {
            if (per_cu >= 4096 * (degree <= 7 ? 2 : 16) && degree <= 12) return {4, 4, win};
            if (per_cu >= 2048 * (degree <= 12 ? 4 : 12) && degree > 7) return {2, 4, win};
        } else if (per_cu >= 2048 * 16) {
            return {2, 4, win};
        }
        choices = {{4, 1, win}, {2, 1, win}, {1, 1, win}};
    } else if (n_t % 16 == 0) choices = {{4, 4, 1u << 17}, {4, 1, 1u << 17}, {2, 1, 1u << 17}, {1, 1, 1u << 17}};
    else if (n_t > 16 && n_t % 4 == 0) choices = {{2, 4, 1u << 15}, {4, 1, 1u << 15}, {2, 1, 1u << 15}, {1, 1, 1u << 15}};
    else if (n_t % 4 == 0) choices = {{4, 1, 1u << 15}, {2, 1, 1u << 15}, {1, 1, 1u << 15}};
    else choices = {{4, 1, 1u << 14}, {2, 1, 1u << 14}, {1, 1, 1u << 14}};
    for (const Layout &l : choices) {
        int64_t tiles = 0;
        for (const ClassInfo &ci : cls) {
            const int64_t span = static_cast<int64_t>(kBlock) * l.qpt * (ci.kind == 2 || ci.kind == 3 ? 1 : l.vq);
            tiles += (ci.count * n_t + span - 1) / span;
        }
        if (tiles >= cus) return l;
    }
    return choices.back();
}

int class_cost(int kind, int degree, int method, int dim) {
    const int ch = dim + (kind != 0 ? 1 : 0);
    if (kind == 2) return 60 + 4 * ch;
    if (kind == 4) {
        const int du = degree >> 4, dv = degree & 15, ncp = (du + 1) * (dv + 1);
        if (method == BZ_DECASTELJAU) return ((du + 1) * dv * (dv + 1) / 2 + du * (du + 1) / 2) * 2 * dim + 8;
        return 3 * (du + dv) + ncp * dim + 8;
    }
    if (kind == 3) return 4 * degree + (degree + 1) * (ch + 2) + 8 + (method == BZ_DECASTELJAU ? degree * (degree + 1) / 2 * ch * 2 : 0);
    if (method == BZ_DECASTELJAU) return degree * (degree + 1) / 2 * ch * 2 + 8;
    return 3 * degree + (degree + 1) * ch + 8;
}

}  // namespace
}  // namespace bzi

using namespace bzi;

struct bz_plan_s {
    int64_t n_obj = 0, n_t = 0;
    int dim = 0, dtype = 0, method = 0;
    // device buffers owned by the plan
    void *ctrl_s = nullptr, *w_s = nullptr;
    int32_t *perm = nullptr;
    Tile *tiles = nullptr;
    NurbsHead *nhead = nullptr;
    uint16_t *ntab = nullptr;
    float *nknots = nullptr;
    void *npts = nullptr;
    bool wide_knots = false;
    unsigned int *counters = nullptr;
    std::vector<ClassInfo> classes;
    std::vector<int32_t> perm_h;  // host copy of perm (window boundaries of the tile order)
    uint32_t n_tiles = 0, n_signed = 0, qpt = 1, vq = 1, window = 0;
    bool has_patches = false;
    int64_t n_segs = 0;
    uint32_t workgroups = 0, cus = 1;
    int dynamic = 1;
};

namespace {

void plan_free(bz_plan_s *p) {
    if (!p) return;
    void *bufs[] = {p->ctrl_s, p->w_s, p->perm, p->tiles, p->nhead, p->ntab, p->nknots, p->npts, p->counters};
    for (void *b : bufs)
        if (b) (void)hipFree(b);
    delete p;
}

// Device copy of a host vector; waits for the copy, so the vector may be
// freed when this returns (plan-time only).
template <typename X>
int dev_upload(X **dst, const std::vector<X> &src, hipStream_t s) {
    const size_t n = std::max<size_t>(src.size(), 1) * sizeof(X);
    hipError_t e = hipMalloc(reinterpret_cast<void **>(dst), n);
    if (e == hipErrorOutOfMemory) return fail(BZ_ERR_NOMEM, "bz_batch_plan_create: device allocation");
    BZ_CHECK_HIP(e);
    if (!src.empty()) {
        BZ_CHECK_HIP(hipMemcpyAsync(*dst, src.data(), src.size() * sizeof(X), hipMemcpyHostToDevice, s));
        BZ_CHECK_HIP(hipStreamSynchronize(s));
    }
    return BZ_OK;
}

int launch_batch(const bz_plan_s *p, const float *t, const float *v, float *out, hipStream_t s, uint32_t workgroups,
                 int dynamic, uint32_t vq) {
    BatchArgs a;
    a.vq = static_cast<int>(vq);
    a.dynamic = dynamic;
    a.ctrl_s = p->ctrl_s;
    a.w_s = p->w_s;
    a.perm = p->perm;
    a.tiles = p->tiles;
    a.n_tiles = p->n_tiles;
    a.n_signed = p->n_signed;
    a.nhead = p->nhead;
    a.ntab = p->ntab;
    a.nknots = p->nknots;
    a.npts = p->npts;
    a.wide_knots = p->wide_knots;
    a.t = t;
    a.v = v;
    a.out = out;
    a.plane = p->n_obj * p->n_t;
    a.n_t = static_cast<uint32_t>(p->n_t);
    a.div_nt = make_fastdiv(a.n_t);
    a.dim = p->dim;
    a.counters = p->counters;
    const bool dc = p->method == BZ_DECASTELJAU;
    workgroups = std::min(workgroups, std::max(1u, p->n_tiles));  // no more than there are tiles
    if (p->dtype == BZ_F32)
        return dc ? launch_batch_kernel<FORM_DC, float>(workgroups, a, s)
                  : launch_batch_kernel<FORM_BERN, float>(workgroups, a, s);
    if (p->dtype == BZ_F16)
        return dc ? launch_batch_kernel<FORM_DC, _Float16>(workgroups, a, s)
                  : launch_batch_kernel<FORM_BERN, _Float16>(workgroups, a, s);
    return dc ? launch_batch_kernel<FORM_DC, bf16_t>(workgroups, a, s)
              : launch_batch_kernel<FORM_BERN, bf16_t>(workgroups, a, s);
}

// Rebuild the tile list for `qpt` sub-tiles of 256 lanes x `vq` queries per
// tile (NURBS tiles one query per lane).  window = 0: class-major order,
// heaviest class first.  window = W: window-major order over consecutive
// blocks of W objects (in the caller's order), and within a window every
// class, heaviest first, for that window's objects -- so the points and
// parameter rows of neighbouring objects, which share cache lines, are
// written and read close together in time.
int build_tiles(bz_plan_s *p, uint32_t qpt, uint32_t vq, uint32_t window, hipStream_t s) {
    const std::vector<ClassInfo> &cls = p->classes;
    std::vector<int> order(cls.size());
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
        return class_cost(cls[x].kind, cls[x].degree, p->method, p->dim) >
               class_cost(cls[y].kind, cls[y].degree, p->method, p->dim);
    });
    std::vector<Tile> tiles;
    auto emit = [&](int c, uint64_t a, uint64_t b) {  // queries [a, b) of class c
        const uint32_t sub = cls[c].kind == 2 ? std::min(qpt, nurbs_sub_tiles(p->dtype == BZ_F32)) : qpt;
        const uint64_t span =
            static_cast<uint64_t>(kBlock) * sub * (cls[c].kind == 0 || cls[c].kind == 1 || cls[c].kind == 4 ? vq : 1);
        for (uint64_t q0 = a; q0 < b; q0 += span)
            tiles.push_back(Tile{cls[c], static_cast<uint32_t>(q0), static_cast<uint32_t>(b), sub, 0});
    };
    const uint64_t nt = static_cast<uint64_t>(p->n_t);
    // signed-weight rational classes (kind 3) go to a launch of their own:
    // their tiles are appended after all others, in class order
    std::vector<int> signed_cls;
    for (int c : order)
        if (cls[c].kind == 3) signed_cls.push_back(c);
    order.erase(std::remove_if(order.begin(), order.end(), [&](int c) { return cls[c].kind == 3; }), order.end());
    if (window == 0) {
        for (int c : order) emit(c, 0, static_cast<uint64_t>(cls[c].count) * nt);
    } else {
        // a class's slots hold its objects in increasing caller order, so the
        // objects of window w are one run of slots per class
        std::vector<int64_t> cur(cls.size(), 0);
        for (int64_t w0 = 0; w0 < p->n_obj; w0 += window) {
            const int32_t w1 = static_cast<int32_t>(std::min<int64_t>(p->n_obj, w0 + window));
            for (int c : order) {
                const int32_t *first = p->perm_h.data() + cls[c].first;
                const int64_t a = cur[c];
                const int64_t b = std::lower_bound(first + a, first + cls[c].count, w1) - first;
                if (b > a) emit(c, static_cast<uint64_t>(a) * nt, static_cast<uint64_t>(b) * nt);
                cur[c] = b;
            }
        }
    }
    // FP32 plans: NURBS tiles, whose queries are chains of dependent loads and take
    // about a sixth of a degree-15 tile's time, fill the launch's end (2^20 curves and
    // 2^16 NURBS x 16: 131 us, 133 spread evenly among the others; with 2^16
    // patches 139 and 152; 2^18 curves and 2^14 NURBS 30 and 40).  16-bit plans
    // have them in their class's place.
    if (p->dtype == BZ_F32)
        std::stable_partition(tiles.begin(), tiles.end(), [](const Tile &t) { return t.ci.kind != 2; });
    const size_t n_main = tiles.size();
    for (int c : signed_cls) emit(c, 0, static_cast<uint64_t>(cls[c].count) * nt);
    if (p->tiles) BZ_CHECK_HIP(hipStreamSynchronize(s));
    if (p->tiles) BZ_CHECK_HIP(hipFree(p->tiles));
    p->tiles = nullptr;
    int rc = dev_upload(&p->tiles, tiles, s);
    if (rc) return rc;
    p->n_tiles = static_cast<uint32_t>(n_main);
    p->n_signed = static_cast<uint32_t>(tiles.size() - n_main);
    p->qpt = qpt;
    p->vq = vq;
    p->window = window;
    return BZ_OK;
}

}  // namespace

extern "C" {

int bz_batch_plan_create(int64_t n_obj, const uint16_t *kind_degree, const int64_t *cp_offset, const void *ctrl,
                         const void *w, int dtype, int dim, const int64_t *knot_offset, const float *knots,
                         int64_t n_t, int method, bz_stream stream, bz_plan *plan) {
    return guarded("bz_batch_plan_create", [&]() -> int {
        const char *fn = "bz_batch_plan_create";
        if (!plan) return fail(BZ_ERR_NULL, "%s: plan is required", fn);
        *plan = nullptr;
        if (n_obj < 0 || n_t < 0) return fail(BZ_ERR_SHAPE, "%s: negative count", fn);
        if (dim < 1 || dim > kMaxDim) return fail(BZ_ERR_SHAPE, "%s: dim %d", fn, dim);
        if (dtype_size(dtype) == 0) return fail(BZ_ERR_DTYPE, "%s: dtype %d", fn, dtype);
        if (method == BZ_AUTO) method = BZ_BERNSTEIN;
        if (method != BZ_DECASTELJAU && method != BZ_BERNSTEIN) return fail(BZ_ERR_UNSUPPORTED, "%s: method %d", fn, method);
        if (n_obj > (int64_t(1) << 31) - 1 || (n_obj > 0 && n_t > ((int64_t(1) << 32) - 1) / std::max<int64_t>(n_obj, 1)))
            return fail(BZ_ERR_SHAPE, "%s: n_obj*n_t must stay below 2^32", fn);
        if (n_obj > 0 && (!kind_degree || !cp_offset || !ctrl))
            return fail(BZ_ERR_NULL, "%s: kind_degree, cp_offset and ctrl are required", fn);
        const hipStream_t s = as_stream(stream);
        std::vector<uint16_t> kd(n_obj);
        std::vector<int64_t> cpo(n_obj + 1, 0), ko;
        if (n_obj > 0) {
            BZ_CHECK_HIP(hipMemcpyAsync(kd.data(), kind_degree, n_obj * sizeof(uint16_t), hipMemcpyDeviceToHost, s));
            BZ_CHECK_HIP(hipMemcpyAsync(cpo.data(), cp_offset, (n_obj + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
            BZ_CHECK_HIP(hipStreamSynchronize(s));
        }
        // validate the objects
        bool need_w = false, any_nurbs = false;
        for (int64_t o = 0; o < n_obj; ++o) {
            const int kind = kd[o] >> 8, deg = kd[o] & 0xff;
            const int64_t ncp = cpo[o + 1] - cpo[o];
            if (kind > 3) return fail(BZ_ERR_SHAPE, "%s: object %lld has kind %d", fn, (long long)o, kind);
            if (kind == 3) {
                const int du = deg >> 4, dv = deg & 15;
                if (du < 1 || du > 3 || dv < 1 || dv > 3)
                    return fail(BZ_ERR_UNSUPPORTED, "%s: patch object %lld has degree (%d, %d) (1..3 each)", fn, (long long)o, du, dv);
                if (ncp != (du + 1) * (dv + 1))
                    return fail(BZ_ERR_SHAPE, "%s: patch object %lld has %lld control points for degree (%d, %d)", fn, (long long)o, (long long)ncp, du, dv);
            } else if (kind == 2) {
                if (deg != kNurbsP) return fail(BZ_ERR_UNSUPPORTED, "%s: NURBS object %lld has degree %d (only cubic)", fn, (long long)o, deg);
                if (ncp < 4) return fail(BZ_ERR_SHAPE, "%s: NURBS object %lld has %lld control points", fn, (long long)o, (long long)ncp);
                any_nurbs = true;
            } else {
                if (deg < 1 || deg > kMaxDegree) return fail(BZ_ERR_SHAPE, "%s: object %lld degree %d", fn, (long long)o, deg);
                if (ncp != deg + 1) return fail(BZ_ERR_SHAPE, "%s: object %lld has %lld control points for degree %d", fn, (long long)o, (long long)ncp, deg);
            }
            if (kind == 1 || kind == 2) need_w = true;
        }
        if (need_w && !w) return fail(BZ_ERR_NULL, "%s: weights are required (rational or NURBS objects)", fn);
        if (!aligned(ctrl, dtype_size(dtype)) || !aligned(w, dtype_size(dtype)))
            return fail(BZ_ERR_ALIGN, "%s: misaligned ctrl or w", fn);
        // which weighted objects have a weight that is not positive
        std::vector<uint8_t> wflag(n_obj, 0);
        if (need_w) {
            uint8_t *flags_d = nullptr;
            hipError_t e = hipMalloc(reinterpret_cast<void **>(&flags_d), std::max<int64_t>(n_obj, 1));
            if (e == hipErrorOutOfMemory) return fail(BZ_ERR_NOMEM, "%s: device allocation", fn);
            BZ_CHECK_HIP(e);
            const uint32_t blocks = static_cast<uint32_t>((n_obj + kBlock - 1) / kBlock);
            if (dtype == BZ_F32)
                hipLaunchKernelGGL((k_weight_flags<float>), dim3(blocks), dim3(kBlock), 0, s, n_obj, kind_degree,
                                   cp_offset, static_cast<const float *>(w), flags_d);
            else if (dtype == BZ_F16)
                hipLaunchKernelGGL((k_weight_flags<_Float16>), dim3(blocks), dim3(kBlock), 0, s, n_obj, kind_degree,
                                   cp_offset, static_cast<const _Float16 *>(w), flags_d);
            else
                hipLaunchKernelGGL((k_weight_flags<bf16_t>), dim3(blocks), dim3(kBlock), 0, s, n_obj, kind_degree,
                                   cp_offset, static_cast<const bf16_t *>(w), flags_d);
            e = hipGetLastError();
            if (e == hipSuccess) e = hipMemcpyAsync(wflag.data(), flags_d, n_obj, hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            (void)hipFree(flags_d);
            if (e != hipSuccess) return hip_fail(e, "k_weight_flags");
        }
        // classes, keyed: 0..14 integral Bezier of degree 1..15, 15..29
        // rational with positive weights, 30..44 rational with a weight <= 0
        // (conditioning test), 45..53 patches of degree (du, dv) in 1..3, 54
        // cubic NURBS (last, so the NURBS rank is its slot in the last class)
        constexpr int kKeys = 55, kPatchKey = 45, kNurbsKey = 54;
        auto key_of = [&](int64_t o) {
            const int kind = kd[o] >> 8, deg = kd[o] & 0xff;
            if (kind == 2) return kNurbsKey;
            if (kind == 3) return kPatchKey + ((deg >> 4) - 1) * 3 + (deg & 15) - 1;
            if (kind == 1 && wflag[o]) return 30 + deg - 1;
            return kind * 15 + deg - 1;
        };
        std::vector<int64_t> count(kKeys, 0);
        for (int64_t o = 0; o < n_obj; ++o) {
            if ((kd[o] >> 8) == 2 && wflag[o])
                return fail(BZ_ERR_UNSUPPORTED, "%s: NURBS object %lld has a weight that is not positive", fn, (long long)o);
            count[key_of(o)] += 1;
        }
        // class list and permutation (stable counting sort by key)
        std::vector<ClassInfo> cls;
        std::vector<int32_t> cls_of_key(kKeys, -1);
        int32_t first = 0;
        int64_t ctrl_elems = 0, w_elems = 0;
        for (int key = 0; key < kKeys; ++key) {
            if (count[key] == 0) continue;
            ClassInfo ci;
            if (key == kNurbsKey) {
                ci.kind = 2;
                ci.degree = kNurbsP;
            } else if (key >= kPatchKey) {
                ci.kind = 4;
                ci.degree = ((key - kPatchKey) / 3 + 1) << 4 | ((key - kPatchKey) % 3 + 1);
            } else {
                ci.kind = key / 15 == 2 ? 3 : key / 15;
                ci.degree = key % 15 + 1;
            }
            ci.first = first;
            ci.count = static_cast<int32_t>(count[key]);
            ci.ctrl_base = ctrl_elems;
            ci.w_base = w_elems;
            if (ci.kind != 2) ctrl_elems += count[key] * class_ncp(ci.kind, ci.degree) * dim;
            if (ci.kind == 1 || ci.kind == 3) w_elems += count[key] * (ci.degree + 1);
            cls_of_key[key] = static_cast<int32_t>(cls.size());
            cls.push_back(ci);
            first += ci.count;
        }
        std::vector<int32_t> perm(n_obj), fill(cls.size(), 0);
        for (int64_t o = 0; o < n_obj; ++o) {
            const int c = cls_of_key[key_of(o)];
            perm[cls[c].first + fill[c]++] = static_cast<int32_t>(o);
        }
        // NURBS (in sorted order, so a NURBS's rank is its slot in the class):
        // read and validate the knot vectors, find the non-empty spans
        std::vector<int64_t> nurbs_obj;
        std::vector<NurbsHead> nhead;
        std::vector<uint16_t> ntab;
        std::vector<float> nknots;
        int64_t n_segs = 0, n_pts = 0;
        bool wide_knots = false;
        if (any_nurbs) {
            if (!knot_offset || !knots) return fail(BZ_ERR_NULL, "%s: knot_offset and knots are required for NURBS", fn);
            ko.resize(n_obj + 1);
            BZ_CHECK_HIP(hipMemcpyAsync(ko.data(), knot_offset, (n_obj + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
            BZ_CHECK_HIP(hipStreamSynchronize(s));
            const int64_t nk_total = ko[n_obj];
            if (nk_total < 0 || nk_total > (int64_t(1) << 34)) return fail(BZ_ERR_SHAPE, "%s: knot_offset", fn);
            std::vector<float> U(nk_total);
            BZ_CHECK_HIP(hipMemcpyAsync(U.data(), knots, nk_total * sizeof(float), hipMemcpyDeviceToHost, s));
            BZ_CHECK_HIP(hipStreamSynchronize(s));
            const ClassInfo &nc = cls.back();
            std::vector<int32_t> spans;
            std::vector<int> buckets;
            for (int32_t r = 0; r < nc.count; ++r) {
                const int64_t o = perm[nc.first + r];
                const int64_t ncp = cpo[o + 1] - cpo[o];
                const int64_t nk = ko[o + 1] - ko[o];
                if (nk != ncp + kNurbsP + 1 || ko[o] < 0 || ko[o + 1] > nk_total)
                    return fail(BZ_ERR_SHAPE, "%s: NURBS object %lld needs %lld knots", fn, (long long)o, (long long)(ncp + 4));
                const float *u = U.data() + ko[o];
                for (int64_t i = 0; i + 1 < nk; ++i)
                    if (!(u[i] <= u[i + 1])) return fail(BZ_ERR_SHAPE, "%s: NURBS object %lld knots not sorted", fn, (long long)o);
                if (u[0] != u[kNurbsP] || u[nk - 1] != u[nk - 1 - kNurbsP] || !(u[kNurbsP] < u[kNurbsP + 1]) ||
                    !(u[nk - 2 - kNurbsP] < u[nk - 1 - kNurbsP]))
                    return fail(BZ_ERR_SHAPE, "%s: NURBS object %lld knot vector is not clamped with end multiplicity 4", fn, (long long)o);
                nurbs_obj.push_back(o);
                spans.clear();
                for (int64_t i = kNurbsP; i < ncp; ++i)
                    if (u[i] < u[i + 1]) spans.push_back(static_cast<int32_t>(i));
                for (int32_t i : spans) wide_knots = wide_knots || knots_wide(u + i - 2);
                if (!add_nurbs(u, ncp, spans, n_pts, nhead, ntab, buckets)) return fail(BZ_ERR_INTERNAL, "%s: NURBS span table", fn);
                nknots.insert(nknots.end(), u, u + nk);
                n_segs += static_cast<int64_t>(spans.size());
                n_pts += ncp;
                if (n_pts > (int64_t(1) << 31) - 1 || ntab.size() > (size_t(1) << 31) - 1)
                    return fail(BZ_ERR_SHAPE, "%s: more than 2^31 NURBS control points", fn);
            }
            nknots.insert(nknots.end(), 4, 0.0f);  // the last NURBS's last window reads one past its knots
        }
        bz_plan_s *p = new (std::nothrow) bz_plan_s();
        if (!p) return fail(BZ_ERR_NOMEM, "%s: host allocation", fn);
        p->n_obj = n_obj;
        p->n_t = n_t;
        p->dim = dim;
        p->dtype = dtype;
        p->method = method;
        p->classes = cls;
        for (const ClassInfo &ci : cls) p->has_patches = p->has_patches || ci.kind == 4;
        p->n_segs = n_segs;
        p->wide_knots = wide_knots;
        const int es = dtype_size(dtype);
        auto dmalloc = [&](void **ptr, size_t bytes) -> int {
            hipError_t e = hipMalloc(ptr, std::max<size_t>(bytes, 16));
            if (e == hipErrorOutOfMemory) return fail(BZ_ERR_NOMEM, "%s: device allocation of %zu bytes", fn, bytes);
            return e == hipSuccess ? BZ_OK : hip_fail(e, "hipMalloc");
        };
        p->perm_h = perm;
        int rc = dev_upload(&p->perm, perm, s);
        if (!rc) rc = dev_upload(&p->nhead, nhead, s);
        if (!rc) rc = dev_upload(&p->ntab, ntab, s);
        if (!rc) rc = dev_upload(&p->nknots, nknots, s);
        if (!rc) {
            int dev = 0, cus = 0;
            hipError_t e = hipGetDevice(&dev);
            if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
            if (e != hipSuccess) rc = hip_fail(e, "device query");
            p->cus = static_cast<uint32_t>(std::max(1, cus));
        }
        if (!rc) {
            const Layout l = default_layout(cls, method, n_t, p->cus);
            rc = build_tiles(p, l.qpt, l.vq, l.window, s);
        }
        if (!rc) rc = dmalloc(&p->ctrl_s, ctrl_elems * es);
        if (!rc) rc = dmalloc(&p->w_s, w_elems * es);
        if (!rc) rc = dmalloc(&p->npts, n_pts * (dim + 1) * es);
        if (!rc) {
            rc = dmalloc(reinterpret_cast<void **>(&p->counters), 2 * sizeof(unsigned int));
            if (!rc && hipMemsetAsync(p->counters, 0, 2 * sizeof(unsigned int), s) != hipSuccess) rc = fail(BZ_ERR_HIP, "%s: memset", fn);
        }
        if (!rc && n_obj > 0) {  // class-sorted copies of control points and weights
            ClassInfo *cls_d = nullptr;
            rc = dev_upload(&cls_d, cls, s);
            if (!rc) {
                const int64_t n_sorted = cls.back().kind == 2 ? cls.back().first : n_obj;
                const uint32_t blocks = static_cast<uint32_t>((n_sorted + kBlock - 1) / kBlock);
                if (n_sorted > 0) {
                    if (es == 4)
                        hipLaunchKernelGGL((k_gather_sorted<uint32_t>), dim3(blocks), dim3(kBlock), 0, s, n_sorted, p->perm,
                                           cp_offset, cls_d, static_cast<int>(cls.size()), dim,
                                           static_cast<const uint32_t *>(ctrl), static_cast<const uint32_t *>(w),
                                           static_cast<uint32_t *>(p->ctrl_s), static_cast<uint32_t *>(p->w_s));
                    else
                        hipLaunchKernelGGL((k_gather_sorted<uint16_t>), dim3(blocks), dim3(kBlock), 0, s, n_sorted, p->perm,
                                           cp_offset, cls_d, static_cast<int>(cls.size()), dim,
                                           static_cast<const uint16_t *>(ctrl), static_cast<const uint16_t *>(w),
                                           static_cast<uint16_t *>(p->ctrl_s), static_cast<uint16_t *>(p->w_s));
                }
                hipError_t e = hipGetLastError();
                if (e == hipSuccess) e = hipStreamSynchronize(s);
                (void)hipFree(cls_d);
                if (e != hipSuccess) rc = hip_fail(e, "k_gather_sorted");
            }
        }
        if (!rc && !nurbs_obj.empty()) {
            int64_t *nobj_d = nullptr;
            rc = dev_upload(&nobj_d, nurbs_obj, s);
            if (!rc) {
                const int nn = static_cast<int>(nurbs_obj.size());
                const uint32_t blocks = (nn + kBlock / 64 - 1) / (kBlock / 64);
                if (es == 4)
                    hipLaunchKernelGGL((k_gather_nurbs<uint32_t>), dim3(blocks), dim3(kBlock), 0, s, nn, nobj_d, cp_offset,
                                       p->nhead, dim, static_cast<const uint32_t *>(ctrl),
                                       static_cast<const uint32_t *>(w), static_cast<uint32_t *>(p->npts));
                else
                    hipLaunchKernelGGL((k_gather_nurbs<uint16_t>), dim3(blocks), dim3(kBlock), 0, s, nn, nobj_d, cp_offset,
                                       p->nhead, dim, static_cast<const uint16_t *>(ctrl),
                                       static_cast<const uint16_t *>(w), static_cast<uint16_t *>(p->npts));
                hipError_t e = hipGetLastError();
                if (e == hipSuccess) e = hipStreamSynchronize(s);
                (void)hipFree(nobj_d);
                if (e != hipSuccess) rc = hip_fail(e, "k_gather_nurbs");
            }
        }
        if (!rc) {
            // default launch: a workgroup per tile (up to 64 per CU), handed out by
            // the hardware as CUs come free: 2^20 curves and 2^16 NURBS x 16, 145 us
            // with 8 workgroups per CU going round the tiles, 138 so (152 and 142
            // with FP16 storage; 500,000 curves: 77 and 76)
            p->workgroups = 64 * p->cus;
            p->dynamic = 0;
        }
        if (!rc) rc = hipStreamSynchronize(s) == hipSuccess ? BZ_OK : fail(BZ_ERR_HIP, "%s: sync", fn);
        if (rc) {
            plan_free(p);
            return rc;
        }
        *plan = p;
        return BZ_OK;
    });
}

static int batch_eval(const char *fn, bz_plan plan, const float *t, const float *v, float *out, bz_stream stream) {
    if (!plan) return fail(BZ_ERR_NULL, "%s: plan is required", fn);
    if (plan->n_obj == 0 || plan->n_t == 0) return BZ_OK;
    if (!t || !out) return fail(BZ_ERR_NULL, "%s: t and out are required", fn);
    if (plan->has_patches && !v)
        return fail(BZ_ERR_NULL, "%s: the plan has surface patches, which need v (bz_batch_eval_uv)", fn);
    if (!aligned(t, 4) || !aligned(v, 4) || !aligned(out, 4)) return fail(BZ_ERR_ALIGN, "%s: misaligned", fn);
    return launch_batch(plan, t, v, out, as_stream(stream), plan->workgroups, plan->dynamic, plan->vq);
}

int bz_batch_eval(bz_plan plan, const float *t, float *out, bz_stream stream) {
    return guarded("bz_batch_eval", [&]() -> int { return batch_eval("bz_batch_eval", plan, t, nullptr, out, stream); });
}

int bz_batch_eval_uv(bz_plan plan, const float *t, const float *v, float *out, bz_stream stream) {
    return guarded("bz_batch_eval_uv",
                   [&]() -> int { return batch_eval("bz_batch_eval_uv", plan, t, v, out, stream); });
}

int bz_batch_plan_autotune(bz_plan plan, const float *t, float *out, bz_stream stream, int64_t *best6) {
    return guarded("bz_batch_plan_autotune", [&]() -> int {
        if (!plan) return fail(BZ_ERR_NULL, "bz_batch_plan_autotune: plan is required");
        if (plan->n_obj == 0 || plan->n_t == 0) return BZ_OK;
        if (!t || !out) return fail(BZ_ERR_NULL, "bz_batch_plan_autotune: t and out are required");
        if (!aligned(t, 4) || !aligned(out, 4)) return fail(BZ_ERR_ALIGN, "bz_batch_plan_autotune: misaligned");
        const hipStream_t s = as_stream(stream);
        hipEvent_t e0, e1;
        BZ_CHECK_HIP(hipEventCreate(&e0));
        BZ_CHECK_HIP(hipEventCreate(&e1));
        const uint32_t cus = plan->cus;
        float best = 0.0f;
        uint32_t best_wg = plan->workgroups, best_q = plan->qpt, best_vq = plan->vq, best_win = plan->window;
        int best_dyn = plan->dynamic;
        const uint32_t qpts[] = {1, 2, 4};
        const uint32_t vqs[] = {1, 4};
        const uint32_t wg_per_cu[] = {8, 12, 16, 64};
        const uint32_t windows[] = {0, 32768, 131072, 262144};
        std::vector<Layout> layouts;
        for (uint32_t win : windows) {
            if (win != 0 && win >= plan->n_obj) continue;  // one window is the class-major order
            for (uint32_t vq : vqs) {
                if (vq == 4 && plan->n_t % 4 != 0) continue;  // four queries of one object per lane
                for (uint32_t q : qpts) layouts.push_back(Layout{q, vq, win});
            }
        }
        // best of three rounds of 5 launches: one round is noisy enough to rank
        // close configurations wrongly.  Patches read their v from t while
        // timing (same size and layout).
        auto time_cfg = [&](uint32_t wg, int dyn, uint32_t vq, float *ms_out) -> int {
            int r0 = launch_batch(plan, t, t, out, s, wg, dyn, vq);  // warm-up
            float ms = 1e30f;
            for (int round = 0; round < 3 && !r0; ++round) {
                BZ_CHECK_HIP(hipEventRecord(e0, s));
                for (int r = 0; r < 5 && !r0; ++r) r0 = launch_batch(plan, t, t, out, s, wg, dyn, vq);
                if (r0) break;
                BZ_CHECK_HIP(hipEventRecord(e1, s));
                BZ_CHECK_HIP(hipEventSynchronize(e1));
                float r_ms = 0;
                BZ_CHECK_HIP(hipEventElapsedTime(&r_ms, e0, e1));
                ms = std::min(ms, r_ms);
            }
            *ms_out = ms;
            return r0;
        };
        // what the plan launches so far first: its layout (the default one of short
        // or odd rows, or a configured one) need not be among those searched (the
        // second timing counts: the first may find the GPU idle)
        int rc = time_cfg(plan->workgroups, plan->dynamic, plan->vq, &best);
        if (!rc) rc = time_cfg(plan->workgroups, plan->dynamic, plan->vq, &best);
        for (const Layout &L : layouts) {
            if (rc) break;
            rc = build_tiles(plan, L.qpt, L.vq, L.window, s);
            for (int dyn = 1; dyn >= 0 && !rc; --dyn)
                for (uint32_t f : wg_per_cu) {
                    float ms = 0;
                    rc = time_cfg(f * cus, dyn, L.vq, &ms);
                    if (rc) break;
                    if (ms < best) {
                        best = ms;
                        best_wg = f * cus;
                        best_q = L.qpt;
                        best_dyn = dyn;
                        best_vq = L.vq;
                        best_win = L.window;
                    }
                }
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        if (rc) return rc;
        rc = build_tiles(plan, best_q, best_vq, best_win, s);
        if (rc) return rc;
        plan->workgroups = best_wg;
        plan->dynamic = best_dyn;
        BZ_CHECK_HIP(hipStreamSynchronize(s));
        if (best6) {
            best6[0] = best_wg;
            best6[1] = best_q;
            best6[2] = static_cast<int64_t>(best * 1000.0f / 5.0f);  // microseconds per launch
            best6[3] = best_dyn;
            best6[4] = best_vq;
            best6[5] = best_win;
        }
        return BZ_OK;
    });
}

int bz_batch_plan_configure(bz_plan plan, int64_t workgroups, int sub_tiles, int schedule, int queries_per_lane,
                            int64_t window, bz_stream stream) {
    return guarded("bz_batch_plan_configure", [&]() -> int {
        const char *fn = "bz_batch_plan_configure";
        if (!plan) return fail(BZ_ERR_NULL, "%s: plan is required", fn);
        if (workgroups < 1 || workgroups > (int64_t(1) << 20)) return fail(BZ_ERR_SHAPE, "%s: workgroups", fn);
        if (sub_tiles != 1 && sub_tiles != 2 && sub_tiles != 4) return fail(BZ_ERR_SHAPE, "%s: sub_tiles", fn);
        if (schedule != 0 && schedule != 1) return fail(BZ_ERR_SHAPE, "%s: schedule", fn);
        if (queries_per_lane != 1 && queries_per_lane != 4) return fail(BZ_ERR_SHAPE, "%s: queries_per_lane", fn);
        if (queries_per_lane == 4 && plan->n_t % 4 != 0)
            return fail(BZ_ERR_UNSUPPORTED, "%s: 4 queries per lane need n_t a multiple of 4", fn);
        if (window < 0 || window > (int64_t(1) << 31) - 1) return fail(BZ_ERR_SHAPE, "%s: window", fn);
        const hipStream_t s = as_stream(stream);
        const int rc = build_tiles(plan, static_cast<uint32_t>(sub_tiles), static_cast<uint32_t>(queries_per_lane),
                                   static_cast<uint32_t>(window), s);
        if (rc) return rc;
        plan->workgroups = static_cast<uint32_t>(workgroups);
        plan->dynamic = schedule;
        BZ_CHECK_HIP(hipStreamSynchronize(s));
        return BZ_OK;
    });
}

int bz_batch_plan_info(bz_plan plan, int64_t *info4) {
    if (!plan || !info4) return fail(BZ_ERR_NULL, "bz_batch_plan_info: plan and info are required");
    info4[0] = static_cast<int64_t>(plan->classes.size());
    info4[1] = plan->n_tiles + plan->n_signed;
    info4[2] = plan->n_segs;
    info4[3] = plan->workgroups;
    return BZ_OK;
}

int bz_plan_destroy(bz_plan plan) {
    return guarded("bz_plan_destroy", [&]() -> int {
        plan_free(plan);
        return BZ_OK;
    });
}

}  // extern "C"
