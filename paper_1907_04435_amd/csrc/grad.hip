// Adjoint of the accrual form with respect to building heights.
//
// The gross shadow of a point over a segment is the measure of the union of
// the occluders' angular intervals, times dt/theta.  Each boundary of that
// union is one end of one occluder's interval; when that end is a crossing
// of the clip line z = H (the ray grazing the roof edge), it moves with the
// height as d(angle)/dH = cross(c, c1 - c0) / (|c|^2 (z1 - z0)) (see
// prism_interval).  So
//     dL/dH_b = sum over points and segments of w * dt/theta *
//               (sum of d(close)/dH - sum of d(open)/dH)
// over the union boundaries owned by b.  The traversal is recomputed here,
// nothing is kept from the forward pass.  Contributions are summed across
// the wave per building and added with one FP64 atomic per building and
// wave into an accumulator (original building ids), which a last kernel
// rounds into the caller's float gradient.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sa_internal.h"
#include "traverse.h"
#include "unit_sched.h"

namespace sa {
namespace {
using namespace dev;

constexpr int kThreads = kSchedThreads;
constexpr int kWaves = kSchedWaves;
constexpr int kSpillBlocks = 1024;

struct GradArgs {
    const float *dl;       // [n_bins * n] or null (all ones)
    double *acc;           // [n_b] FP64 accumulator, original ids
    const int32_t *order;  // hierarchy position -> original id
};

template <bool kBlocks>
__device__ __forceinline__ void grad_segment(const ViewEntry *view, int n_b, cint *voff, TileFan *tile, cfloat4 *verts, cfloat *height,
                                             const SegConst &g, const LanePoint &q, bool active,
                                             float w0, float w1, UnionG &U, bool &ov)
{
    union_clear(U);
    ov = false;
    float W0u, W0v, W1u, W1v;
    window_dirs(g, w0, w1, W0u, W0v, W1u, W1v);
    bool live = active;
    if (active && q.own >= 0) {
        float a, b;
        if (backface_interval(q.nx, q.ny, g, w0, w1, W0u, W0v, W1u, W1v, a, b)) {
            union_first(U, a, b, -1, -1, 0.f, 0.f);
            live = !(a <= w0 && b >= w1);
        }
    }
    if (view == nullptr) return;
    uint64_t ovm = 0;
    auto leaf = [&](int prim, int voff, int m, uint64_t want) -> uint64_t {
        const uint64_t gm = want & ballot(prim != q.own);
        if (!gm) return 0;
        float a, b, da, db;
        const uint64_t hit = prism_interval<true>(verts, voff, m, ld(height + prim), gm, q.px, q.py, q.pz, g, w0, w1,
                                                  W0u, W0v, W1u, W1v, a, b, da, db);
        if (!hit) return 0;
        const uint64_t over = union_insert_mask(U, a, b, prim, da, db, hit);
        ovm |= over;
        // the whole window is shadowed: no boundary inside it
        return over | (hit & ballot(U.n == 1 && U.lo[0] <= w0 && U.hi[0] >= w1));
    };
    const SegFan ft(g, q.px, q.py, q.pz);
    Work none{0, 0, 0, 0, 0, 0, 0};
    walk_view<false, kBlocks>(view, n_b, voff, tile, ballot(live), ft, leaf, none);
    ov = lane_in(ovm);
}

// Add v into acc[order[prim]] for every lane with prim >= 0.  Lanes that
// hold the same building are summed across the wave first (a fixed
// butterfly order), then one lane issues a single FP64 atomic: one atomic
// per building and wave instead of one per lane.  Must be reached by every
// lane of the wave (the shuffles read all lanes).
__device__ __forceinline__ void wave_scatter(int prim, double v, const GradArgs &G)
{
    const int lane = tid() & 63;
    uint64_t pend = ballot(prim >= 0);
    while (pend) {
        const int lead = __builtin_ctzll(pend);
        const int key = __shfl(prim, lead, 64);
        const uint64_t m = pend & ballot(prim == key);
        double sum = lane_in(m) ? v : 0.0;
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == lead) atomicAdd(&G.acc[G.order[key]], sum);
        pend &= ~m;
    }
}

// The union boundaries of one lane's window that move with a height:
// closing ends +, opening ends -, each times wscale; ok = false adds
// nothing (every lane of the wave must call this).
__device__ __forceinline__ void scatter_grad(const UnionG &U, bool ok, float wscale, const GradArgs &G)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool in = ok && r < U.n;
        if (!ballot(in)) break;  // no lane's set is this large
        wave_scatter(in && U.plo[r] >= 0 && U.dlo[r] != 0.f ? U.plo[r] : -1, -(double)(wscale * U.dlo[r]), G);
        wave_scatter(in && U.phi[r] >= 0 && U.dhi[r] != 0.f ? U.phi[r] : -1, (double)(wscale * U.dhi[r]), G);
    }
}

// Six waves per SIMD: at seven (72 VGPRs) the interval sets with their owners
// spill 87 registers, at five there are too few waves (forward and adjoint on
// 200k points, 1-minute knots: 10.77, 10.15 and 10.69 ms at 7, 6 and 5).
// Persistent: its units are (tile, every n-th segment), enough of them to
// keep every wave busy on small point sets (the gradient sums are atomic, so
// any split adds up the same).
template <bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_grad(
    RoofBoxes B, const ViewEntry *views_g, int n_b, const int32_t *voff_g, const float4 *verts_g,
    const float *height_g, const SegConst *segs_g, int j0, int j1, Sched W, PointArgs P, GradArgs G, SpillArgs S)
{
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSeg *segs = (cSeg *)segs_g;
    __shared__ int s_B[sizeof(RoofBoxes) / 4];
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    __shared__ int s_G[sizeof(GradArgs) / 4];
    __shared__ int s_S[sizeof(SpillArgs) / 4];
    if (tid() == 0) {
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        lds_park((lds_int *)s_B, B);
        lds_park((lds_int *)s_G, G);
        lds_park((lds_int *)s_S, S);
    }
    __syncthreads();
    __shared__ TileFan s_tile[kWaves];
    TileFan *tile = &s_tile[tid() >> 6];
    const int lane = tid() & 63;
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, j0, j1, kx, un)) {
        const int ja = uniform(un.a), jb = uniform(un.b), step = uniform(un.step);
        const PointArgs Pd = lds_uniform<PointArgs>((lds_int *)s_P);
        const uint32_t i = un.tile * 64u + (uint32_t)lane;  // (fewer than 2^31 points)
        const bool valid = i < Pd.n;
        const LanePoint q = load_point(Pd, i, valid);
        const bool covered = roof_covered<kBlocks>(lds_uniform<RoofBoxes>((lds_int *)s_B), (cint *)voff_g, verts, height, q, valid);
        int bin = -1;
        float w = 0.f;
        for (int j = ja; j < jb; j += step) {
            const SegConst g = ld(segs + j);
            if (g.bin != bin) {
                bin = g.bin;
                const GradArgs Gd = lds_uniform<GradArgs>((lds_int *)s_G);
                w = (valid && Gd.dl) ? Gd.dl[(int64_t)bin * Pd.n + i] : 1.f;
            }
            UnionG U;
            bool ov;
            const ViewEntry *view = views_g ? views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all : nullptr;
            grad_segment<kBlocks>(view, n_b, (cint *)voff_g, tile, verts, height, g, q, valid && !covered && w != 0.f, 0.f, g.theta,
                         U, ov);
            scatter_grad(U, valid && !covered && !ov && w != 0.f, w * g.wrate, lds_uniform<GradArgs>((lds_int *)s_G));
            const uint64_t over = ballot(valid && ov);
            if (over) spill_push(lds_uniform<SpillArgs>((lds_int *)s_S), over, (int)i, j);
        }
    }
}

// The adjoint's spilled point-segments: as the accrual form's, one wave each,
// every lane one 64th of the window, sub-windows split again.  Ends clamped to
// a sub-window do not move with a height, so splitting adds no gradient terms.
template <bool kBlocks>
__global__ __launch_bounds__(kThreads) void k_grad_spill(const ViewEntry *views_g, int n_b, int j0,
                                                         const int32_t *voff_g, const float4 *verts_g,
                                                         const float *height_g, const SegConst *segs_g, PointArgs P,
                                                         GradArgs G, const int4 *queue, uint32_t *counters, int32_t cap)
{
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSeg *segs = (cSeg *)segs_g;
    __shared__ SpillWindow s_wait[kWaves][kSpillWait];
    SpillWindow *wait = s_wait[tid() >> 6];
    __shared__ TileFan s_tile[kWaves];
    TileFan *tile = &s_tile[tid() >> 6];
    const int lane = tid() & 63;
    uint32_t singles;
    const int64_t total = spill_items(counters, cap, singles), stride = (int64_t)n_wg() * kWaves;
    for (int64_t t = (int64_t)wg_id() * kWaves + (tid() >> 6); t < total; t += stride) {
        int j;
        const int64_t i = spill_item(queue, singles, t, j);
        if (i < 0) continue;
        const LanePoint q = load_point(P, i, true);
        const SegConst g = ld(segs + j);
        const float w = G.dl ? G.dl[(int64_t)g.bin * P.n + i] : 1.f;
        const ViewEntry *view = views_g ? views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all : nullptr;
        SpillWindow win{0.f, g.theta, 0};
        for (int waiting = 0;;) {
            float w0, w1;
            spill_share(win, lane, w0, w1);
            UnionG U;
            bool ov;
            grad_segment<kBlocks>(view, n_b, (cint *)voff_g, tile, verts, height, g, q, true, w0, w1, U, ov);
            scatter_grad(U, !ov, w * g.wrate, G);
            if (!spill_next(wait, waiting, ov, w0, w1, counters + 2, win)) break;
        }
    }
}

// grad[b] = (add ? grad[b] : 0) + scale * acc[b], rounded once to float.
__global__ void k_grad_out(const double *acc, int32_t n_b, double scale, int add, float *grad)
{
    const int b = wg_id() * wg_size() + tid();
    if (b < n_b) grad[b] = (float)((add ? (double)grad[b] : 0.0) + scale * acc[b]);
}

}  // namespace

sa_status launch_grad(const DeviceScene &s, const DevicePath &p, const PointsView &pts, const float *dl, float scale,
                      bool add, float *grad, const TileLaunch &L, SpillQueue &q, Scratch &scr, Scratch &acc_scr,
                      hipStream_t st, std::string &err)
{
    if (s.n_b == 0) return SA_OK;
    const size_t need = sizeof(double) * (size_t)s.n_b;
    if (!reserve(acc_scr, need, st)) {
        err = "no room for the gradient accumulator (under stream capture an eager call of the size comes first)";
        return SA_ERR_OOM;
    }
    double *acc = (double *)acc_scr.ptr;
    sa_status rc = fill_u32(acc, 2 * (int64_t)s.n_b, 0u, st, err);
    if (rc != SA_OK) return rc;
    int64_t tiles;
    if (!tile_count(pts.n, tiles, err)) return SA_ERR_INVALID_ARG;
    const auto kern = has_blocks(s.n_b) ? k_grad<true> : k_grad<false>;
    const int64_t res = resident_blocks(kern, L);
    const PointArgs P{pts.n, pts.x, pts.y, pts.z, pts.nx, pts.ny, pts.owner, s.rank, s.n_b};
    const GradArgs G{dl, acc, s.order};
    // segment ranges whose per-segment views fit the budget, each
    // followed by its spilled windows
    const int64_t per = std::min(std::max<int64_t>(1, kSpillWork / std::max<int64_t>(64 * tiles, 1)), seg_views_cap(s, p, scr, st));
    for (int64_t j0 = 0; pts.n > 0 && j0 < p.n_segs; j0 += per) {
        const int j1 = (int)std::min<int64_t>(j0 + per, p.n_segs);
        ViewEntry *views;
        rc = build_seg_views(s, p.segs, s.height, (int)j0, j1, scr, {q.counters, q.grab, 8 * kGrabStride}, st, views, err);
        if (rc != SA_OK) return rc;
        SpillArgs S{q.entries, q.counters, q.capacity};
        const Sched W = plan_units(p.seg_runs, (int)j0, j1, tiles, Split::kChunks, res, q.grab);
        hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0, st, RoofBoxes{s.pbox, s.gbox, s.vorder, s.n_b, 0}, views,
                           s.n_b, s.voff, s.verts, s.height, p.segs, (int)j0, j1, W, P, G, S);
        hipLaunchKernelGGL(has_blocks(s.n_b) ? k_grad_spill<true> : k_grad_spill<false>, dim3(kSpillBlocks), dim3(kThreads), 0, st, views, s.n_b, (int)j0, s.voff,
                           s.verts, s.height, p.segs, P, G, (const int4 *)q.entries, q.counters, q.capacity);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            err = std::string("gradient kernels: ") + hipGetErrorString(e);
            return SA_ERR_DEVICE;
        }
    }
    hipLaunchKernelGGL(k_grad_out, dim3((unsigned)((s.n_b + 255) / 256)), dim3(256), 0, st, (const double *)acc,
                       s.n_b, (double)scale, add ? 1 : 0, grad);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        err = std::string("gradient output: ") + hipGetErrorString(e);
        return SA_ERR_DEVICE;
    }
    return SA_OK;
}

}  // namespace sa
