// Gross-shadow kernels: the sampled form (one shadow ray per point per sun
// instant) and the accrual form (one occluded interval per occluder per
// point per great-circle segment, union, measure), plus the accrual spill
// rounds that finish the rare point-segments whose occluded set has more
// than four disjoint pieces by splitting their window 64 ways.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sa_internal.h"
#include "traverse.h"
#include "unit_sched.h"
#include "views.h"

namespace sa {
namespace {
using namespace dev;

constexpr int kThreads = kSchedThreads;
constexpr int kWaves = kSchedWaves;
constexpr int kSpillBlocks = 1536;  // six of k_spill on each of 256 CUs (1,024: block scene 6.78 ms, so 6.65)
constexpr int64_t kChunkWork = 2000000000ll;  // point-segments per contribution launch
// Views per launch.  A launch has its set-up, its spilled
// windows and a last unit that others wait for: a year on 45,000 prisms and
// 500,000 points takes 236, 219 and 207 ms in launches of 150, 300 and 600
// segments (views of 256, 512 and 1024 MiB then, of half as much now).  Where that much cannot be had, down to kLeastViewBytes.
constexpr int64_t kViewBytes = 1024ll << 20;
constexpr int64_t kLeastViewBytes = 256ll << 20;
constexpr int64_t kPieceBytes = 256ll << 20;    // per-piece sums of an accrual launch on few tiles

// Per-bin outputs of the accrual kernels.  A bin whose first segment lies in
// the launch is stored (no clear beforehand, no read); a bin continued from
// an earlier launch, or any bin under SA_FLAG_ADD, is added to.  Each
// (tile, bin) belongs to one unit, so the sums are deterministic.  With
// pieces (pcnt non-null) a unit holds one piece of a bin's run instead and
// writes its sums to its part's row of pcnt / pmin ([part][n]); a second
// kernel adds a bin's pieces in order into the outputs.
struct BinOut {
    int32_t *counts;
    float *minutes;
    double *minutes64;    // the FP64 lane sums behind minutes (optional)
    int32_t *pcnt;        // per-piece sums, or null
    double *pmin;
    int32_t fresh_first;  // the launch's first bin starts in it
    int32_t fresh_rest;   // the later bins of the launch start in it
    float scale;          // minutes are multiplied by this
    int32_t pad;
};

__device__ __forceinline__ void put_bin(const BinOut &O, int64_t o, bool fresh, int cnt, double mins)
{
    const double v = mins * O.scale;
    if (O.counts) O.counts[o] = (fresh ? 0 : O.counts[o]) + cnt;
    if (O.minutes) O.minutes[o] = (fresh ? 0.f : O.minutes[o]) + (float)v;
    if (O.minutes64) O.minutes64[o] = (fresh ? 0.0 : O.minutes64[o]) + v;
}

// ------------------------------------------------------------------ sampled
// Outputs of the sampled form (parked in LDS by the kernel).
struct SampOut {
    int32_t *counts;
    float *minutes;
    uint32_t *bits;
    float *longest;
    float scale;
    int32_t pad;
};

// Adds a unit's sums for one bin (outputs cleared beforehand; a bin of a
// tile belongs to one unit).
__device__ __forceinline__ void sampled_put(const SampOut &O, int64_t o, int cnt, float mins, float best)
{
    if (O.counts) O.counts[o] += cnt;
    if (O.minutes) O.minutes[o] += mins * O.scale;
    if (O.longest) O.longest[o] = fmaxf(O.longest[o], best * O.scale);
}

// The sampled form: an any-hit ray per (point, instant), in packets of
// 64 / kInst neighbouring points x kInst consecutive instants of one
// 64-point tile (kInst is a launch choice; 16 x 4 on the block scene).  A
// packet first takes the back-face test and the occluder cache: each wave
// remembers the prism that blocked the most lanes of its previous walk and
// tests it first; a blocked ray is blocked whichever prism is found first,
// so the predicate is unchanged.  The rays left go to a per-wave queue in
// LDS as (instant, point of the group), and a walk of the hierarchy runs
// whenever 64 are queued, and once more for the rest at the end of the
// point group.  A packet enters the queue with about four rays in five
// live (block scene: the rest face away from their facade or are blocked
// by the cached occluder), while every node visit costs the wave the same
// whatever its live lanes; refilled walks are full.  The queue fills in the
// order of the instants, so a walk holds the group's points at neighbouring
// instants.  Eight waves per SIMD (the compiler's own choice gives seven).
//
// k_sampled_q: counts and minutes of units that lie in one bin; a walk's
// hits add their instant's weight to their point's sum in LDS.
template <bool kCount, int kInst>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_sampled_q(
    const Node *nodes_g, const float4 *verts_g, const float *height_g, const SampleConst *samples_g, int K, Sched W,
    PointArgs P, SampOut O, uint64_t *work)
{
    static_assert(kInst >= 1 && kInst <= 16 && (kInst & (kInst - 1)) == 0, "instants per packet");
    constexpr int kPts = 64 / kInst;  // points per packet (a group)
    constexpr int kQueue = 128;       // < 64 waiting plus one packet
    Work wk{0, 0, 0, 0, 0, 0, 0};
    cNode *nodes = (cNode *)nodes_g;
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSample *samples = (cSample *)samples_g;
    __shared__ StackEntry s_stack[kWaves][kStackDepth];
    __shared__ uint32_t s_queue[kWaves][kQueue];
    __shared__ int s_cnt[kWaves][kPts];
    __shared__ float s_min[kWaves][kPts];
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    __shared__ int s_O[sizeof(SampOut) / 4];
    if (tid() == 0) {
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        lds_park((lds_int *)s_O, O);
    }
    __syncthreads();
    const int wave = tid() >> 6;
    StackEntry *stack = s_stack[wave];
    uint32_t *queue = s_queue[wave];
    int *g_cnt = s_cnt[wave];
    float *g_min = s_min[wave];
    const int lane = tid() & 63;
    const int slot = lane & (kInst - 1);  // the lane's instant within the packet
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, 0, K, kx, un)) {
        const int ka = uniform(un.a), kb = uniform(un.b);
        if (kb <= ka) continue;
        const int64_t n = lds_uniform<PointArgs>((lds_int *)s_P).n;
        const int bin = ld(samples + ka).tag & kBinMask;
        for (int g = 0; g < kInst; ++g) {
            const int64_t i0 = (int64_t)un.tile * 64 + g * kPts;  // the group's first point
            if (i0 >= n) break;
            if (lane < kPts) {
                g_cnt[lane] = 0;
                g_min[lane] = 0.f;
            }
            int c_prim = -1, c_voff = 0, c_m = 0;  // the occluder cache
            int queued = 0;
            // one walk over the first nq queued rays; lanes past nq idle
            auto walk = [&](int nq) {
                const bool on = lane < nq;
                const uint32_t e = on ? queue[lane] : 0u;
                const int pt = (int)(e & 63u);
                const SampleConst s = samples_g[on ? (int)(e >> 6) : ka];
                // the middle ray's direction orders the children
                const SampleConst sm = ld(samples + uniform((int)(queue[nq >> 1] >> 6)));
                const LanePoint q = load_point(lds_uniform<PointArgs>((lds_int *)s_P), i0 + pt, on);
                uint64_t hitm = 0;
                int b_prim = -1, b_voff = 0, b_m = 0, b_cnt = 0;
                const float ox = -q.px * s.ix, oy = -q.py * s.iy, oz = -q.pz * s.iz;
                auto bt = [&](float x0, float y0, float x1, float y1, float z1) {
                    const float ax = fmaf(x0, s.ix, ox), bx = fmaf(x1, s.ix, ox);
                    const float ay = fmaf(y0, s.iy, oy), by = fmaf(y1, s.iy, oy);
                    const float tfz = fmaf(z1, s.iz, oz);
                    const float tn = fmaxf(fmaxf(fminf(ax, bx), fminf(ay, by)), 0.f);
                    const float tf = fminf(fminf(fmaxf(ax, bx), fmaxf(ay, by)), tfz);
                    return le_mask(tn, tf);
                };
                auto leaf = [&](int prim, int voff, int m, uint64_t want) -> uint64_t {
                    const bool go = lane_in(want & ballot(prim != q.own));
                    if constexpr (kCount) {
                        wk.prism += go ? 1u : 0u;
                        wk.edges += go ? (uint32_t)m : 0u;
                        wk.leaves += first_active_lane() ? 1u : 0u;
                    }
                    const bool t =
                        go & ray_prism(verts, voff, m, ld(height + prim), q.px, q.py, q.pz, s.dx, s.dy, s.dz);
                    const uint64_t tm = ballot(t);
                    hitm |= tm;
                    const int cn = __builtin_popcountll(tm);
                    if (cn > b_cnt) {
                        b_cnt = cn;
                        b_prim = prim;
                        b_voff = voff;
                        b_m = m;
                    }
                    return tm;  // a blocked ray needs no further test
                };
                auto key = [&](float x0, float y0, float x1, float y1, float z1) {
                    return fmaf(x0 + x1, sm.dx, fmaf(y0 + y1, sm.dy, z1 * sm.dz));
                };
                packet_traverse<kCount>(nodes, stack, ballot(on), bt, leaf, key, wk);
                c_prim = uniform(b_cnt > 0 ? b_prim : -1);
                c_voff = uniform(b_voff);
                c_m = uniform(b_m);
                if (lane_in(hitm)) {
                    atomicAdd(&g_cnt[pt], 1);
                    atomicAdd(&g_min[pt], s.w);
                }
            };
            const int64_t i = i0 + lane / kInst;
            const bool pvalid = i < n;
            const LanePoint q = load_point(lds_uniform<PointArgs>((lds_int *)s_P), pvalid ? i : 0, pvalid);
            int cnt = 0;  // this lane's instants settled before any walk
            float mins = 0.f;
            for (int c0 = ka; c0 < kb; c0 += kInst) {
                const int k = c0 + slot;
                const bool valid = pvalid && k < kb;
                const SampleConst s = samples_g[k < kb ? k : ka];
                const bool back = q.own >= 0 && fmaf(q.nx, s.dx, q.ny * s.dy) <= 0.f;
                uint64_t live = ballot(valid && !back);
                uint64_t cached = 0;
                if (nodes_g != nullptr && c_prim >= 0 && live) {
                    const bool go = lane_in(live & ballot(c_prim != q.own));
                    if constexpr (kCount) {
                        wk.prism += go ? 1u : 0u;
                        wk.edges += go ? (uint32_t)c_m : 0u;
                        wk.leaves += first_active_lane() ? 1u : 0u;
                    }
                    cached = ballot(go & ray_prism(verts, c_voff, c_m, ld(height + c_prim), q.px, q.py, q.pz, s.dx,
                                                   s.dy, s.dz));
                    live &= ~cached;
                }
                if constexpr (kCount) wk.units += valid ? 1u : 0u;
                const bool sh = valid && (back || lane_in(cached));
                cnt += sh ? 1 : 0;
                mins += sh ? s.w : 0.f;
                if (nodes_g != nullptr && live) {
                    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
                    if (lane_in(live)) queue[queued + rank] = ((uint32_t)k << 6) | (uint32_t)(lane / kInst);
                    queued += __builtin_popcountll(live);
                    if (queued >= 64) {
                        walk(64);
                        // the rest (fewer than 64) to the front
                        const bool more = 64 + lane < queued;
                        const uint32_t e = more ? queue[64 + lane] : 0u;
                        if (more) queue[lane] = e;
                        queued -= 64;
                    }
                }
            }
            if (queued > 0) walk(queued);
            // the point's lanes together, then its walks' hits
            for (int o = 1; o < kInst; o <<= 1) {
                cnt += __shfl_xor(cnt, o, 64);
                mins += __shfl_xor(mins, o, 64);
            }
            if (slot == 0 && pvalid) {
                const int pt = lane / kInst;
                sampled_put(lds_uniform<SampOut>((lds_int *)s_O), (int64_t)bin * n + i, cnt + g_cnt[pt],
                            mins + g_min[pt], 0.f);
            }
        }
    }
    if constexpr (kCount) flush_work(wk, work);
}

// k_sampled_qb: the outputs that need every instant's result -- bit
// vectors, the continuous shadow (in time order), and bins that interleave
// (a unit then spans them).  The instants of a unit go in windows of kWin
// (a 2 KB bitmap per wave: 256 instants for 64 points, up to 4096 for 4):
// each window's packets and walks set their shadowed (point, instant)
// pairs in a per-wave LDS bitmap, the queue is drained at the window's
// end, and each point's lane then replays the window's bits in time order:
// counts, minutes and runs per bin, a run reset at each day's first instant
// (runs never cross days) and the longest kept per bin.  A queue entry
// holds the instant's offset in the window, so any path length fits.  With
// bit vectors a unit is a whole tile from the first instant, so windows
// start on 32-instant words and the bitmap words are the output words.
template <bool kCount, int kInst>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_sampled_qb(
    const Node *nodes_g, const float4 *verts_g, const float *height_g, const SampleConst *samples_g, int K, Sched W,
    PointArgs P, SampOut O, uint64_t *work)
{
    static_assert(kInst >= 1 && kInst <= 16 && (kInst & (kInst - 1)) == 0, "instants per packet");
    constexpr int kPts = 64 / kInst;  // points per packet (a group)
    constexpr int kQueue = 128;       // < 64 waiting plus one packet
    constexpr int kWords = 512 / kPts;  // bitmap words per point and window (2 KB a wave)
    constexpr int kWin = 32 * kWords;   // instants per window
    constexpr int kRow = kWords + 1;    // a point's row, padded: lanes reading one word of
                                        // consecutive points hit different banks
    Work wk{0, 0, 0, 0, 0, 0, 0};
    cNode *nodes = (cNode *)nodes_g;
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSample *samples = (cSample *)samples_g;
    __shared__ StackEntry s_stack[kWaves][kStackDepth];
    __shared__ uint32_t s_queue[kWaves][kQueue];
    __shared__ uint32_t s_map[kWaves][kPts * kRow];
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    __shared__ int s_O[sizeof(SampOut) / 4];
    if (tid() == 0) {
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        lds_park((lds_int *)s_O, O);
    }
    __syncthreads();
    const int wave = tid() >> 6;
    StackEntry *stack = s_stack[wave];
    uint32_t *queue = s_queue[wave];
    uint32_t *map = s_map[wave];
    const int lane = tid() & 63;
    const int slot = lane & (kInst - 1);  // the lane's instant within the packet
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, 0, K, kx, un)) {
        const int ka = uniform(un.a), kb = uniform(un.b);
        if (kb <= ka) continue;
        const int64_t n = lds_uniform<PointArgs>((lds_int *)s_P).n;
        for (int g = 0; g < kInst; ++g) {
            const int64_t i0 = (int64_t)un.tile * 64 + g * kPts;  // the group's first point
            if (i0 >= n) break;
            const int64_t i = i0 + lane / kInst;
            const bool pvalid = i < n;
            const LanePoint q = load_point(lds_uniform<PointArgs>((lds_int *)s_P), pvalid ? i : 0, pvalid);
            // replay state of point `lane` of the group (lanes < kPts)
            const bool rvalid = lane < kPts && i0 + lane < n;
            int cnt = 0;
            float mins = 0.f, run = 0.f, best = 0.f;
            int bin = ld(samples + ka).tag & kBinMask;
            int c_prim = -1, c_voff = 0, c_m = 0;  // the occluder cache
            for (int w0 = ka; w0 < kb; w0 += kWin) {
                const int w1 = min(w0 + kWin, kb);
                for (int t = lane; t < kPts * kRow; t += 64) map[t] = 0u;
                int queued = 0;
                // one walk over the first nq queued rays; lanes past nq idle
                auto walk = [&](int nq) {
                    const bool on = lane < nq;
                    const uint32_t e = on ? queue[lane] : 0u;
                    const int pt = (int)(e & 63u), j = (int)(e >> 6);
                    const SampleConst s = samples_g[on ? w0 + j : ka];
                    // the middle ray's direction orders the children
                    const SampleConst sm = ld(samples + w0 + uniform((int)(queue[nq >> 1] >> 6)));
                    const LanePoint qw = load_point(lds_uniform<PointArgs>((lds_int *)s_P), i0 + pt, on);
                    uint64_t hitm = 0;
                    int b_prim = -1, b_voff = 0, b_m = 0, b_cnt = 0;
                    const float ox = -qw.px * s.ix, oy = -qw.py * s.iy, oz = -qw.pz * s.iz;
                    auto bt = [&](float x0, float y0, float x1, float y1, float z1) {
                        const float ax = fmaf(x0, s.ix, ox), bx = fmaf(x1, s.ix, ox);
                        const float ay = fmaf(y0, s.iy, oy), by = fmaf(y1, s.iy, oy);
                        const float tfz = fmaf(z1, s.iz, oz);
                        const float tn = fmaxf(fmaxf(fminf(ax, bx), fminf(ay, by)), 0.f);
                        const float tf = fminf(fminf(fmaxf(ax, bx), fmaxf(ay, by)), tfz);
                        return le_mask(tn, tf);
                    };
                    auto leaf = [&](int prim, int voff, int m, uint64_t want) -> uint64_t {
                        const bool go = lane_in(want & ballot(prim != qw.own));
                        if constexpr (kCount) {
                            wk.prism += go ? 1u : 0u;
                            wk.edges += go ? (uint32_t)m : 0u;
                            wk.leaves += first_active_lane() ? 1u : 0u;
                        }
                        const bool t = go & ray_prism(verts, voff, m, ld(height + prim), qw.px, qw.py, qw.pz, s.dx,
                                                      s.dy, s.dz);
                        const uint64_t tm = ballot(t);
                        hitm |= tm;
                        const int cn = __builtin_popcountll(tm);
                        if (cn > b_cnt) {
                            b_cnt = cn;
                            b_prim = prim;
                            b_voff = voff;
                            b_m = m;
                        }
                        return tm;  // a blocked ray needs no further test
                    };
                    auto key = [&](float x0, float y0, float x1, float y1, float z1) {
                        return fmaf(x0 + x1, sm.dx, fmaf(y0 + y1, sm.dy, z1 * sm.dz));
                    };
                    packet_traverse<kCount>(nodes, stack, ballot(on), bt, leaf, key, wk);
                    c_prim = uniform(b_cnt > 0 ? b_prim : -1);
                    c_voff = uniform(b_voff);
                    c_m = uniform(b_m);
                    if (lane_in(hitm)) atomicOr(&map[pt * kRow + (j >> 5)], 1u << (j & 31));
                };
                for (int c0 = w0; c0 < w1; c0 += kInst) {
                    const int k = c0 + slot;
                    const bool valid = pvalid && k < w1;
                    const SampleConst s = samples_g[k < w1 ? k : ka];
                    const bool back = q.own >= 0 && fmaf(q.nx, s.dx, q.ny * s.dy) <= 0.f;
                    uint64_t live = ballot(valid && !back);
                    uint64_t cached = 0;
                    if (nodes_g != nullptr && c_prim >= 0 && live) {
                        const bool go = lane_in(live & ballot(c_prim != q.own));
                        if constexpr (kCount) {
                            wk.prism += go ? 1u : 0u;
                            wk.edges += go ? (uint32_t)c_m : 0u;
                            wk.leaves += first_active_lane() ? 1u : 0u;
                        }
                        cached = ballot(go & ray_prism(verts, c_voff, c_m, ld(height + c_prim), q.px, q.py, q.pz,
                                                       s.dx, s.dy, s.dz));
                        live &= ~cached;
                    }
                    if constexpr (kCount) wk.units += valid ? 1u : 0u;
                    const int pt = lane / kInst, j = k - w0;
                    if (valid && (back || lane_in(cached))) atomicOr(&map[pt * kRow + (j >> 5)], 1u << (j & 31));
                    if (nodes_g != nullptr && live) {
                        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
                        if (lane_in(live)) queue[queued + rank] = ((uint32_t)j << 6) | (uint32_t)pt;
                        queued += __builtin_popcountll(live);
                        if (queued >= 64) {
                            walk(64);
                            // the rest (fewer than 64) to the front
                            const bool more = 64 + lane < queued;
                            const uint32_t e = more ? queue[64 + lane] : 0u;
                            if (more) queue[lane] = e;
                            queued -= 64;
                        }
                    }
                }
                if (queued > 0) walk(queued);
                // the window's bitmap words are the output words
                uint32_t *bits = lds_uniform<SampOut>((lds_int *)s_O).bits;
                if (bits != nullptr)
                    for (int t = lane; t < kPts * kWords; t += 64) {
                        const int wd = t / kPts, p = t - wd * kPts;  // consecutive lanes: consecutive points
                        if (i0 + p < n && w0 + 32 * wd < w1)
                            bits[(int64_t)((w0 >> 5) + wd) * n + i0 + p] = map[p * kRow + wd];
                    }
                // replay in time order, one point per lane
                for (int wd = 0; wd < kWords && w0 + 32 * wd < w1; ++wd) {
                    const uint32_t word = rvalid ? map[lane * kRow + wd] : 0u;
                    const int jb = min(32, w1 - w0 - 32 * wd);
                    for (int b = 0; b < jb; ++b) {
                        const SampleConst sj = ld(samples + (w0 + 32 * wd + b));
                        const int sbin = sj.tag & kBinMask;
                        if (sbin != bin) {
                            if (rvalid)
                                sampled_put(lds_uniform<SampOut>((lds_int *)s_O), (int64_t)bin * n + i0 + lane, cnt,
                                            mins, best);
                            cnt = 0;
                            mins = 0.f;
                            best = 0.f;
                            bin = sbin;
                        }
                        if (sj.tag & kDayStart) run = 0.f;
                        const bool sh = (word >> b) & 1u;
                        cnt += sh ? 1 : 0;
                        mins += sh ? sj.w : 0.f;
                        run = sh ? run + sj.w : 0.f;
                        best = fmaxf(best, run);
                    }
                }
            }
            if (rvalid) sampled_put(lds_uniform<SampOut>((lds_int *)s_O), (int64_t)bin * n + i0 + lane, cnt, mins, best);
        }
    }
    if constexpr (kCount) flush_work(wk, work);
}

// ------------------------------------------------------------------ accrual
// Segment j's constants read again where they are used after a traversal
// rather than held in registers across it (an opaque copy of the index
// keeps the compiler from reusing the first load): a scalar-cache hit
// costs less than spilling them to lanes of a vector register.
__device__ __forceinline__ SegConst reload(cSeg *segs, int j)
{
    int jr = j;
    asm volatile("" : "+s"(jr));
    return ld(segs + jr);
}

// Measure and sample count of the occluded set of one point over the
// window [w0, w1] of segment g.  `last_window` says whether w1 is the end
// of the segment (instants at the window end belong to the next window
// otherwise).
__device__ __forceinline__ void measure(const Union4 &U, const SegConst &g, float w0, float w1,
                                        bool last_window, double &mins, int &cnt)
{
    const float scale = g.rate;
    float m = 0.f;
    int c = 0;
    const float inv_step = g.inv_step;
    int kmax = g.ns - 1;
    if (!last_window) kmax = min(kmax, (int)ceilf((w1 * scale - g.s0) * inv_step) - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (!ballot(r < U.n)) break;  // no lane's set is this large
        if (r < U.n) {
            m += U.hi[r] - U.lo[r];
            const int klo = max((int)ceilf((U.lo[r] * scale - g.s0) * inv_step), 0);
            // a set that reaches the window end holds the window's last
            // instant: taken as is, not through the rounding of w1 * scale
            const int khi = U.hi[r] >= w1 ? kmax : min((int)floorf((U.hi[r] * scale - g.s0) * inv_step), kmax);
            c += max(khi - klo + 1, 0);
        }
    }
    mins += (double)(m * g.wrate);
    cnt += c * g.mult;
}

// The scene as the current segment sees it, the vertex offsets of the leaves,
// and the heights.
struct SegSrc {
    const ViewEntry *view;
    int n_b;
    cint *voff;
    TileFan *tile;  // the wave's slot
    cfloat *height;
};

// The occluded set of every active lane's point over its window of segment g:
// back-face term, then the walk of the view (which takes the whole wave).  On
// return `ov` marks lanes whose set needed more than four pieces.
template <bool kCount, bool kBlocks>
__device__ __forceinline__ void accrue_segment(const SegSrc &src, cfloat4 *verts, const SegConst &g, const LanePoint &q,
                                               bool active, float w0, float w1, Union4 &U, bool &ov, Work &wk)
{
    union_clear(U);
    ov = false;
    float W0u, W0v, W1u, W1v;
    window_dirs(g, w0, w1, W0u, W0v, W1u, W1v);
    bool live = active;
    if (active && q.own >= 0) {
        float a, b;
        if (backface_interval(q.nx, q.ny, g, w0, w1, W0u, W0v, W1u, W1v, a, b)) {
            union_first(U, a, b);
            live = !(a <= w0 && b >= w1);
        }
    }
    if (src.view == nullptr) return;
    // liveness and overflow as wave masks (see walk_view)
    uint64_t ovm = 0;
    auto leaf = [&](int prim, int voff, int m, uint64_t want) -> uint64_t {
        const uint64_t gm = want & ballot(prim != q.own);
        if (!gm) return 0;
        if constexpr (kCount) {
            wk.prism += lane_in(gm) ? 1u : 0u;
            wk.edges += lane_in(gm) ? (uint32_t)m : 0u;
            wk.leaves += first_active_lane() ? 1u : 0u;
        }
        float a, b, da, db;
        const float H = ld(src.height + prim);
        const uint64_t hit = prism_interval<false>(verts, voff, m, H, gm, q.px, q.py, q.pz, g, w0, w1, W0u, W0v, W1u,
                                                   W1v, a, b, da, db);
        if constexpr (kCount) wk.inserts += lane_in(hit) ? 1u : 0u;
        if (!hit) return 0;
        const uint64_t over = union_insert_mask(U, a, b, hit);
        ovm |= over;
        // the whole window is in shadow
        return over | (hit & ballot(U.n == 1 && U.lo[0] <= w0 && U.hi[0] >= w1));
    };
    const SegFan ft(g, q.px, q.py, q.pz);
    walk_view<kCount, kBlocks>(src.view, src.n_b, src.voff, src.tile, ballot(live), ft, leaf, wk);
    ov = lane_in(ovm);
}

__global__ void k_clear_state(LaunchState L) { clear_state(L, tid()); }

// kOcc waves per SIMD, a launch choice (6, 7 or 8; the tuner measures
// them).  At 8 the kernel fits in 64 VGPRs (the compiler would settle for
// fewer waves otherwise), which hides more of the scalar-load and
// compare-chain latency of the traversal loop.
template <bool kCount, int kOcc, bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kOcc))) void k_accrual(
    RoofBoxes B, const ViewEntry *views_g, int n_b, const int32_t *voff_g, const float4 *verts_g,
    const float *height_g, const SegConst *segs_g, int j0, int j1, Sched W, PointArgs P, BinOut O, SpillArgs S,
    uint64_t *work)
{
    Work wk{0, 0, 0, 0, 0, 0, 0};
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSeg *segs = (cSeg *)segs_g;
    __shared__ int s_B[sizeof(RoofBoxes) / 4];
    // the outputs are needed only when a bin ends, the schedule once per
    // unit: parked in LDS so their pointers hold no scalar registers
    // through the traversal loop
    __shared__ int s_O[sizeof(BinOut) / 4];
    __shared__ int s_S[sizeof(SpillArgs) / 4];
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    if (tid() == 0) {
        lds_park((lds_int *)s_O, O);
        lds_park((lds_int *)s_S, S);
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        lds_park((lds_int *)s_B, B);
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
        const int64_t n = Pd.n;
        const int64_t i = (int64_t)un.tile * 64 + lane;
        const bool valid = i < n;
        const LanePoint q = load_point(Pd, i, valid);
        const bool covered = roof_covered<kBlocks>(lds_uniform<RoofBoxes>((lds_int *)s_B), (cint *)voff_g, verts, height, q, valid);

        int cnt = 0;
        double mins = 0.0;  // per-lane FP64: long spans sum thousands of segment measures
        int bin = jb > ja ? ld(segs + ja).bin : 0;
        const BinOut O0 = lds_uniform<BinOut>((lds_int *)s_O);
        bool fresh = (ja == j0 ? O0.fresh_first : O0.fresh_rest) != 0;
        for (int j = ja; j < jb; j += step) {
            const SegConst g = ld(segs + j);
            if (g.bin != bin) {
                const BinOut Ob = lds_uniform<BinOut>((lds_int *)s_O);
                if (valid) put_bin(Ob, (int64_t)bin * n + i, fresh, cnt, mins);
                cnt = 0;
                mins = 0.0;
                bin = g.bin;
                fresh = Ob.fresh_rest != 0;
            }
            Union4 U;
            bool ov;
            const SegSrc src{views_g ? views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all : nullptr, n_b, (cint *)voff_g,
                             tile, height};
            accrue_segment<kCount, kBlocks>(src, verts, g, q, valid && !covered, 0.f, g.theta, U, ov, wk);
            if constexpr (kCount) {
                wk.units += valid ? 1u : 0u;
                wk.spills += (valid && ov) ? 1u : 0u;
            }
            const SegConst gm = reload(segs, j);
            if (covered && valid) {
                mins += (double)gm.dt;
                cnt += gm.ns_all;
            } else if (!ov) {
                measure(U, gm, 0.f, gm.theta, true, mins, cnt);
            }
            const uint64_t over = ballot(valid && ov);
            if (over) spill_push(lds_uniform<SpillArgs>((lds_int *)s_S), over, (int)i, j);
        }
        const BinOut Oe = lds_uniform<BinOut>((lds_int *)s_O);
        if (Oe.pcnt) {
            // a piece of one bin's run: its sums go to the part's row
            if (valid) {
                Oe.pcnt[(int64_t)un.part * n + i] = cnt;
                Oe.pmin[(int64_t)un.part * n + i] = mins;
            }
        } else if (valid && jb > ja) {
            put_bin(Oe, (int64_t)bin * n + i, fresh, cnt, mins);
        }
    }
    if constexpr (kCount) flush_work(wk, work);
}

// Adds the pieces of every run of a launch, in piece order, into the run's
// bin: the launch's first run is stored or added to as O says for the
// launch's first bin, the others as for its later bins.
// One point and run (r0 + the y index) per thread.  A round trip to rows that other
// XCDs have just written takes 2 us, so 24 rows are asked for at once, the
// run's bin beside them (16,384 points, 20 rows: 9.3 -> 4.7 us).
constexpr int kRowsInFlight = 24;

__global__ __launch_bounds__(64) void k_add_pieces(Sched W, int r0, int j0, const SegConst *__restrict__ segs, int64_t n,
                                                   BinOut O, const int64_t *__restrict__ var_off, int V)
{
    const int sub = W.sub > 1 ? W.sub : 1;
    const int r = r0 + wg_id_y();
    const int64_t i = (int64_t)wg_id() * 64 + tid();
    if (i >= n) return;
    if (var_off && (i < var_off[0] || i >= var_off[V])) return;  // no variant's point
    int cnt = 0;
    double mins = 0.0;
    for (int p0 = r * sub; p0 < (r + 1) * sub; p0 += kRowsInFlight) {
        int c[kRowsInFlight];
        double m[kRowsInFlight];
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) {
            const int64_t row = (int64_t)min(p0 + u, (r + 1) * sub - 1) * n + i;
            c[u] = O.pcnt[row];
            m[u] = O.pmin[row];
        }
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) {
            const bool in = p0 + u < (r + 1) * sub;
            cnt += in ? c[u] : 0;
            mins += in ? m[u] : 0.0;
        }
    }
    const int bin = segs[max(W.part_start[r], j0)].bin;
    put_bin(O, (int64_t)bin * n + i, (r == 0 ? O.fresh_first : O.fresh_rest) != 0, cnt, mins);
}

// Continuous shadow (Sec. 3.1) over one window [w0, w1] whose occluded set
// U is sorted and disjoint: a set that starts at w0 extends the current run
// (the run so far reached the window start), any gap ends it; best keeps
// the longest run in minutes.  Applied window after window in time order
// this joins the per-segment prefix, longest and suffix as Sec. 6 stitches
// them across the edges of a day's path.
__device__ __forceinline__ void runs_update(const Union4 &U, float w0, float w1, float rate, float &run, float &best)
{
    if (U.n == 0) run = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (r < U.n) {
            const float len = (U.hi[r] - U.lo[r]) * rate;
            run = (r == 0 && U.lo[0] <= w0) ? run + len : len;
            best = fmaxf(best, run);
            if (U.hi[r] < w1) run = 0.f;
        }
    }
}

// The accrual form with the continuous shadow of every point.  Runs must be
// followed in time order, so a segment whose set needs more than four
// pieces is not queued as a spilled window: the lane walks that segment
// window by window from its start (halving the window on overflow,
// doubling it after a success) while the other lanes wait.  A window would
// have to shrink below theta / 4096 to raise the overflow flag.  Seven
// waves per SIMD (the compiler fits the kernel in 72 VGPRs) measured 4 %
// faster than the six its natural allocation allows.
template <bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(7))) void k_accrual_runs(
    RoofBoxes B, const ViewEntry *views_g, int n_b, const int32_t *voff_g, const float4 *verts_g,
    const float *height_g, const SegConst *segs_g, int j0, int j1, Sched W, PointArgs P, BinOut O, float *longest,
    uint32_t *overflow)
{
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSeg *segs = (cSeg *)segs_g;
    __shared__ int s_B[sizeof(RoofBoxes) / 4];
    // outputs (and where to flag overflow), schedule and points parked in
    // LDS: needed once per unit or at a bin's end, they hold no scalar
    // registers through the traversal
    __shared__ int s_O[sizeof(BinOut) / 4];
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    __shared__ float *s_longest;
    __shared__ uint32_t *s_overflow;
    if (tid() == 0) {
        lds_park((lds_int *)s_O, O);
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        lds_park((lds_int *)s_B, B);
        s_longest = longest;
        s_overflow = overflow;
    }
    __syncthreads();
    __shared__ TileFan s_tile[kWaves];
    TileFan *tile = &s_tile[tid() >> 6];
    const int lane = tid() & 63;
    Work none{0, 0, 0, 0, 0, 0, 0};
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, j0, j1, kx, un)) {
        const PointArgs Pd = lds_uniform<PointArgs>((lds_int *)s_P);
        const int64_t n = Pd.n;
        const int64_t i = (int64_t)un.tile * 64 + lane;
        const bool valid = i < n;
        const LanePoint q = load_point(Pd, i, valid);
        const bool covered = roof_covered<kBlocks>(lds_uniform<RoofBoxes>((lds_int *)s_B), (cint *)voff_g, verts, height, q, valid);
        const int ja = uniform(un.a), jb = uniform(un.b);

        int cnt = 0;
        double mins = 0.0;
        float run = 0.f, best = 0.f;
        int bin = jb > ja ? ld(segs + ja).bin : 0;
        int day = jb > ja ? ld(segs + ja).day : 0;
        const BinOut O0 = lds_uniform<BinOut>((lds_int *)s_O);
        bool fresh = (ja == j0 ? O0.fresh_first : O0.fresh_rest) != 0;
        auto flush = [&]() {
            if (!valid) return;
            const int64_t o = (int64_t)bin * n + i;
            const BinOut Ob = lds_uniform<BinOut>((lds_int *)s_O);
            put_bin(Ob, o, fresh, cnt, mins);
            float *lg = s_longest;
            if (lg) lg[o] = fresh ? best * Ob.scale : fmaxf(lg[o], best * Ob.scale);
        };
        for (int j = ja; j < jb; ++j) {
            const SegConst g = ld(segs + j);
            if (g.bin != bin) {
                flush();
                cnt = 0;
                mins = 0.0;
                best = 0.f;
                bin = g.bin;
                fresh = lds_uniform<BinOut>((lds_int *)s_O).fresh_rest != 0;
            }
            if (g.day != day) {
                run = 0.f;
                day = g.day;
            }
            if (covered && valid) {
                mins += (double)g.dt;
                cnt += g.ns_all;
                run += g.dt;
                best = fmaxf(best, run);
            }
            bool pending = valid && !covered;
            float w0 = 0.f, s = g.theta;
            while (ballot(pending)) {
                const float w1 = fminf(w0 + s, g.theta);
                Union4 U;
                bool ov;
                const SegSrc src{views_g ? views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all : nullptr, n_b,
                                 (cint *)voff_g, tile, height};
                accrue_segment<false, kBlocks>(src, verts, g, q, pending, w0, w1, U, ov, none);
                if (pending) {
                    if (ov) {
                        if (s < g.theta * (1.0f / 4096.0f)) {
                            atomicOr(s_overflow, 2u);
                            pending = false;
                        } else {
                            s *= 0.5f;
                        }
                    } else {
                        const SegConst gm = reload(segs, j);
                        measure(U, gm, w0, w1, w1 >= gm.theta, mins, cnt);
                        runs_update(U, w0, w1, gm.rate, run, best);
                        w0 = w1;
                        pending = w0 < g.theta;
                        s = fminf(2.f * s, g.theta);
                    }
                }
            }
        }
        if (jb > ja) flush();
    }
}

// The queued point-segments: each is taken by one wave whose 64 lanes take
// one 64th of the window each.  Every lane follows the same point along the
// same segment, so the wave's traversal stays coherent (a lane per queued
// entry would walk 64 unrelated points).  Sub-windows that still need more
// than four pieces wait in LDS and are split 64 ways again, three levels in
// all (1/262144 of a segment; what is left then raises the overflow flag).
// The lanes' measures are summed across the wave and added with one atomic
// per output.  One launch: as three rounds over two queues, with their
// clears, it was seven (4 us each and the gaps where nothing is queued).
template <bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_spill(
    const ViewEntry *views_g, int n_b, int j0, const int32_t *voff_g, const float4 *verts_g, const float *height_g,
    const SegConst *segs_g, PointArgs P, float scale, int32_t *counts, float *minutes, double *minutes64,
    const int4 *queue, uint32_t *counters, int32_t cap)
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
        const SegSrc src{views_g ? views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all : nullptr, n_b, (cint *)voff_g,
                         tile, height};
        SpillWindow win{0.f, g.theta, 0};
        double mins = 0.0;
        int cnt = 0;
        for (int waiting = 0;;) {
            float w0, w1;
            spill_share(win, lane, w0, w1);
            Union4 U;
            bool ov;
            Work none{0, 0, 0, 0, 0, 0, 0};
            accrue_segment<false, kBlocks>(src, verts, g, q, true, w0, w1, U, ov, none);
            if (!ov) measure(U, g, w0, w1, w1 >= g.theta, mins, cnt);
            if (!spill_next(wait, waiting, ov, w0, w1, counters + 2, win)) break;
        }
        for (int o = 32; o > 0; o >>= 1) {
            mins += __shfl_xor(mins, o, 64);
            cnt += __shfl_xor(cnt, o, 64);
        }
        if (lane == 0) {
            const int64_t o = (int64_t)g.bin * P.n + i;
            if (minutes) atomicAdd(&minutes[o], (float)(mins * scale));
            if (minutes64) atomicAdd(&minutes64[o], mins * scale);
            if (counts) atomicAdd(&counts[o], cnt);
        }
    }
}

// ------------------------------------------------------------------ contribution
// Building contribution (Sec. 7.2): every building's own occluded interval
// over each segment, never merged with the others' and with no early exit
// (a lane whose window is already shadowed keeps walking: later buildings
// still count).  The lanes' weighted minutes for one leaf are summed across
// the wave and added with one FP64 atomic; a back-facing wall counts for
// the point's own building.  Eight waves per SIMD (56 VGPRs): 17.5 ms on
// the block scene against 19.4 at the compiler's seven.
template <bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_contrib(const ViewEntry *views_g, int n_b, const int32_t *voff_g,
                                                      const float4 *verts_g, const float *height_g,
                                                      const SegConst *segs_g, int j0, int j1, Sched W, PointArgs P,
                                                      const float *weight, const int32_t *order,
                                                      double *contrib)
{
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cSeg *segs = (cSeg *)segs_g;
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    if (tid() == 0) {
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
    }
    __syncthreads();
    __shared__ TileFan s_tile[kWaves];
    TileFan *tile = &s_tile[tid() >> 6];
    const int lane = tid() & 63;
    Work none{0, 0, 0, 0, 0, 0, 0};
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, j0, j1, kx, un)) {
        const PointArgs Pd = lds_uniform<PointArgs>((lds_int *)s_P);
        const int64_t i = (int64_t)un.tile * 64 + lane;
        const bool valid = i < Pd.n;
        const LanePoint q = load_point(Pd, i, valid);
        const float wt = valid ? (weight ? weight[i] : 1.f) : 0.f;
        const bool active = valid & (wt != 0.f);
        // Back-facing minutes go to the point's own building: kept per lane
        // over the bin's segments and added once per bin, with one atomic
        // for the wave when all its contributing lanes share the building
        // (facade points come wall by wall, so they nearly always do).
        const int ja = uniform(un.a), jb = uniform(un.b), step = uniform(un.step);
        double bf = 0.0;
        int bin = jb > ja ? ld(segs + ja).bin : 0;
        // Sums of the bin by building: lane l holds the one of a building with
        // rank l modulo 64, until another takes its place or the bin ends.  An
        // atomic per leaf before: waves of an XCD meet the same few buildings
        // at the same time, and their adds to one word queue up (600 prisms
        // and 20,000 points 226 -> 190 us, 60,000 points 420 -> 379; 5,000
        // prisms and 300,000 points 1,089 -> 1,065).
        int key = -1;
        double held = 0.0;
        auto flush_held = [&]() {
            if (key >= 0) atomicAdd(contrib + (int64_t)bin * n_b + order[key], held);
            key = -1;
        };
        auto flush_backface = [&]() {
            const uint64_t has = ballot(bf != 0.0);
            if (!has) return;
            const int lead = (int)__builtin_ctzll(has);
            const int o0 = __shfl(q.own, lead, 64);
            double *row = contrib + (int64_t)bin * n_b;
            if (!ballot(bf != 0.0 && q.own != o0)) {
                double s = bf;
                for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
                if (lane == lead) atomicAdd(&row[order[o0]], s);
            } else if (bf != 0.0) {
                atomicAdd(&row[order[q.own]], bf);
            }
            bf = 0.0;
        };
        for (int j = ja; j < jb; j += step) {
            const SegConst g = ld(segs + j);
            if (g.bin != bin) {
                flush_held();
                flush_backface();
                bin = g.bin;
            }
            if (active && q.own >= 0) {
                float a, b;
                if (backface_interval(q.nx, q.ny, g, 0.f, g.theta, 1.f, 0.f, g.cth, g.sth, a, b))
                    bf += (double)((b - a) * g.wrate * wt);
            }
            if (views_g == nullptr) continue;
            const SegFan ft(g, q.px, q.py, q.pz);
            auto leaf = [&](int prim, int voff, int m, uint64_t want) -> uint64_t {
                const uint64_t gm = want & ballot(prim != q.own);
                if (!gm) return 0;
                float a, b, da, db;
                const uint64_t hit = prism_interval<false>(verts, voff, m, ld(height + prim), gm, q.px, q.py, q.pz, g, 0.f,
                                                           g.theta, 1.f, 0.f, g.cth, g.sth, a, b, da, db);
                if (!hit) return 0;
                // the wave's total for this building (every lane is active
                // here: the traversal runs on the whole wave)
                const float v = wave_sum(lane_in(hit) ? (b - a) * g.wrate * wt : 0.f);
                if (lane == (prim & 63)) {
                    if (key != prim) {
                        flush_held();
                        key = prim;
                        held = 0.0;
                    }
                    held += (double)v;
                }
                return 0;  // no lane retires: every building counts
            };
            walk_view<false, kBlocks>(views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all, n_b, (cint *)voff_g, tile, ballot(active),
                             ft, leaf, none);
        }
        flush_held();
        flush_backface();
    }
}

// ------------------------------------------------------------------ batched
// Variant v of the scene differs from the base only in the heights of a few
// buildings.  One set of views serves them all: it is built for the tallest a
// prism is in any of them, so a walk passes every prism that meets a point's
// fan in its variant (boxes only decide what is tested), and the leaf takes
// the variant's own height.

// Heights of the variants (the base's), the greatest of each prism (the
// base's) and the tile offsets: tile_off[v] = first tile of variant v, 64
// points per tile.
__global__ void k_var_copy(const float *__restrict__ base_h, int n_b, int V, float *__restrict__ vh, float *__restrict__ tops,
                           const int64_t *__restrict__ var_off, int64_t *__restrict__ tile_off)
{
    const int64_t stride = (int64_t)n_wg() * wg_size();
    const int64_t t0 = (int64_t)wg_id() * wg_size() + tid();
    for (int64_t t = t0; t < (int64_t)V * n_b; t += stride) vh[t] = base_h[t % n_b];
    for (int64_t t = t0; t < n_b; t += stride) tops[t] = base_h[t];
    if (t0 < 64) {  // one wave, 64 variants at a time
        int64_t base = 0;
        for (int v0 = 0; v0 < V; v0 += 64) {
            const int v = v0 + (int)t0;
            int64_t sum = v < V ? (var_off[v + 1] - var_off[v] + 63) / 64 : 0;
            const int64_t own = sum;
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t up = __shfl_up(sum, o, 64);
                sum += (int)t0 >= o ? up : 0;
            }
            if (v < V) tile_off[v] = base + sum - own;
            base += __shfl(sum, 63, 64);
        }
        if (t0 == 0) tile_off[V] = base;
    }
}

// The variants' heights, bad ones skipped and flagged; a thread each.  (Heights
// are positive, so their order is that of their bits.)
__global__ void k_var_heights(int64_t n, int k, const int32_t *__restrict__ ids, const float *__restrict__ h,
                              const int32_t *__restrict__ rank, int n_b, float *__restrict__ vh, int32_t *tops, uint32_t *flag)
{
    const int64_t t = (int64_t)wg_id() * wg_size() + tid();
    if (t >= n) return;
    const int id = ids[t];
    const float hv = h[t];
    if (id < 0 || id >= n_b || !(hv > 0.f)) {
        atomicOr(flag, 4u);
        return;
    }
    const int prim = rank[id];
    vh[t / k * n_b + prim] = hv;
    atomicMax(&tops[prim], __float_as_int(hv));
}

// The accrual form over the variants' tiles, in units as k_accrual's: tile t
// is variant v's (t - tile_off[v])-th, found by binary search (the launch has
// as many tiles as there could be; those past the last are empty).  A
// point-segment whose occluded set needs more than four pieces is finished in
// place by walking its window left to right with halving / doubling
// sub-windows.  Seven waves per SIMD: 72 VGPRs with a few spilled to scratch,
// measured faster than eight (2.39 and 2.46 ms on 32 variants of 1M points) and
// no slower than six.  Whole tiles as units before, drawn from one counter: 32
// variants of 1M points on 20,000 prisms took 2.37 ms, in (tile, bin) units
// 1.70; 40 of 60,000 points on 3,000 prisms 1.05, in pieces 0.25; 5 of 300,000
// on 400 prisms 1.51 and 0.67.
template <bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(7))) void k_batched(
    RoofBoxes B, const ViewEntry *views_g, int n_b, const int32_t *voff_g, const float4 *verts_g,
    const float *vh_g, const SegConst *segs_g, int j0, int j1, Sched W, PointArgs P, BinOut O,
    const int64_t *__restrict__ var_off, const int64_t *__restrict__ tile_off, int V, uint32_t *flag)
{
    cfloat4 *verts = (cfloat4 *)verts_g;
    cSeg *segs = (cSeg *)segs_g;
    __shared__ int s_B[sizeof(RoofBoxes) / 4];
    __shared__ int s_O[sizeof(BinOut) / 4];
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    __shared__ TileFan s_tile[kWaves];
    if (tid() == 0) {
        lds_park((lds_int *)s_O, O);
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        lds_park((lds_int *)s_B, B);
    }
    __syncthreads();
    TileFan *tile = &s_tile[tid() >> 6];
    const int lane = tid() & 63;
    Work none{0, 0, 0, 0, 0, 0, 0};
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, j0, j1, kx, un)) {
        const int64_t t = un.tile;
        if (t >= tile_off[V]) continue;
        int lo = 0, hi = V - 1;  // last v with tile_off[v] <= t
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tile_off[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const int v = uniform(lo);
        const int ja = uniform(un.a), jb = uniform(un.b), step = uniform(un.step);
        cfloat *height = (cfloat *)(vh_g + (int64_t)v * n_b);
        const PointArgs Pd = lds_uniform<PointArgs>((lds_int *)s_P);
        const int64_t n = Pd.n;
        const int64_t i = var_off[v] + (t - tile_off[v]) * 64 + lane;
        const bool valid = i < var_off[v + 1];
        const LanePoint q = load_point(Pd, i, valid);
        const bool covered = roof_covered<kBlocks>(lds_uniform<RoofBoxes>((lds_int *)s_B), (cint *)voff_g, verts, height, q, valid);
        int cnt = 0;
        double mins = 0.0;
        int bin = jb > ja ? ld(segs + ja).bin : 0;
        for (int j = ja; j < jb; j += step) {
            const SegConst g = ld(segs + j);
            if (g.bin != bin) {
                if (valid) put_bin(lds_uniform<BinOut>((lds_int *)s_O), (int64_t)bin * n + i, false, cnt, mins);
                cnt = 0;
                mins = 0.0;
                bin = g.bin;
            }
            if (covered && valid) {
                mins += (double)g.dt;
                cnt += g.ns_all;
            }
            float w0 = 0.f, s = g.theta;
            bool pending = valid && !covered;
            while (ballot(pending)) {
                const float w1 = fminf(w0 + s, g.theta);
                Union4 U;
                bool ov;
                const SegSrc src{views_g ? views_g + (int64_t)(j - j0) * view_shape<kBlocks>(n_b).all : nullptr, n_b,
                                 (cint *)voff_g, tile, height};
                accrue_segment<false, kBlocks>(src, verts, g, q, pending, w0, w1, U, ov, none);
                if (pending) {
                    if (ov) {
                        if (s < g.theta * (1.0f / 4096.0f)) {
                            atomicOr(flag, 2u);
                            pending = false;
                        } else {
                            s *= 0.5f;
                        }
                    } else {
                        measure(U, reload(segs, j), w0, w1, w1 >= g.theta, mins, cnt);
                        w0 = w1;
                        pending = w0 < g.theta;
                        s = fminf(2.f * s, g.theta);
                    }
                }
            }
        }
        const BinOut Oe = lds_uniform<BinOut>((lds_int *)s_O);
        if (Oe.pcnt) {
            // a piece of one bin's run: its sums go to the part's row
            if (valid) {
                Oe.pcnt[(int64_t)un.part * n + i] = cnt;
                Oe.pmin[(int64_t)un.part * n + i] = mins;
            }
        } else if (valid && jb > ja) {
            put_bin(Oe, (int64_t)bin * n + i, false, cnt, mins);
        }
    }
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    const int64_t stride = (int64_t)n_wg() * wg_size();
    for (int64_t t = (int64_t)wg_id() * wg_size() + tid(); t < n; t += stride) p[t] = v;
}

}  // namespace

#define SA_CHECK_LAUNCH(what)                                                   \
    do {                                                                        \
        hipError_t e_ = hipGetLastError();                                      \
        if (e_ != hipSuccess) {                                                 \
            err = std::string(what) + ": " + hipGetErrorString(e_);             \
            return SA_ERR_DEVICE;                                               \
        }                                                                       \
    } while (0)

// Parts of n points whose sums the scratch has room for.  Asked for in one
// size, whatever the call: no call then frees what a graph captured over
// another holds, and one under capture finds what an eager one left.
static int64_t piece_parts(Scratch &scr, int64_t n, hipStream_t st)
{
    (void)reserve_wish(scr, (size_t)kPieceBytes + 256, st);
    const int64_t per_part = n * (int64_t)(sizeof(int32_t) + sizeof(double));
    return std::max<int64_t>(0, (int64_t)scr.bytes - 256) / per_part;
}

// k_add_pieces over a launch's runs, as many at a time as a grid has rows.
static void add_pieces(const Sched &W, int j0, const DevicePath &p, int64_t n, const BinOut &O, const int64_t *var_off,
                       int n_var, hipStream_t st)
{
    constexpr int kRows = 32768;
    const int runs = (int)W.n_parts / W.sub;
    for (int r0 = 0; r0 < runs; r0 += kRows)
        hipLaunchKernelGGL(k_add_pieces, dim3((unsigned)((n + 63) / 64), (unsigned)std::min(kRows, runs - r0)), dim3(64), 0,
                           st, W, r0, j0, (const SegConst *)p.segs, n, O, var_off, n_var);
}

static RoofBoxes roof_boxes(const DeviceScene &s) { return RoofBoxes{s.pbox, s.gbox, s.vorder, s.n_b, 0}; }

static PointArgs point_args(const PointsView &pts, const DeviceScene &s)
{
    return PointArgs{pts.n, pts.x, pts.y, pts.z, pts.nx, pts.ny, pts.owner, s.rank, s.n_b};
}

sa_status launch_sampled(const DeviceScene &s, const DevicePath &p, const PointsView &pts, float scale,
                         int32_t *counts, float *minutes, uint32_t *bits, float *longest, uint64_t *work,
                         const TileLaunch &L, uint32_t *grab, hipStream_t st, std::string &err)
{
    if (pts.n == 0) return SA_OK;
    int64_t tiles;
    if (!tile_count(pts.n, tiles, err)) return SA_ERR_INVALID_ARG;
    const Node *nodes = s.n_b > 0 ? s.nodes : nullptr;
    const int ni = L.sampled_instants;
    // Counts and minutes of units that lie in one bin: the queue with the
    // points' sums in LDS (its entries hold the instant, below 2^26).  Bit
    // vectors, the continuous shadow and bins that interleave: the queue
    // with a bitmap replayed in time order; bit vectors pack 32 instants a
    // word across bin boundaries, so a unit is then a whole tile and each
    // word has one writer.
    auto kern = work ? k_sampled_qb<true, 8> : k_sampled_qb<false, 8>;
    if (ni == 1) kern = work ? k_sampled_qb<true, 1> : k_sampled_qb<false, 1>;
    if (ni == 2) kern = work ? k_sampled_qb<true, 2> : k_sampled_qb<false, 2>;
    if (ni == 4) kern = work ? k_sampled_qb<true, 4> : k_sampled_qb<false, 4>;
    if (ni == 16) kern = work ? k_sampled_qb<true, 16> : k_sampled_qb<false, 16>;
    const Split split = bits ? Split::kNone : Split::kUniqueBins;
    int64_t res = resident_blocks(kern, L);
    Sched W = plan_units(p.sample_runs, 0, p.n_samples, tiles, split, res, grab);
    if (!bits && !longest && p.n_samples < (1 << 26) &&
        (W.part_start != nullptr || p.sample_runs.start.size() == 2)) {
        kern = work ? k_sampled_q<true, 8> : k_sampled_q<false, 8>;
        if (ni == 1) kern = work ? k_sampled_q<true, 1> : k_sampled_q<false, 1>;
        if (ni == 2) kern = work ? k_sampled_q<true, 2> : k_sampled_q<false, 2>;
        if (ni == 4) kern = work ? k_sampled_q<true, 4> : k_sampled_q<false, 4>;
        if (ni == 16) kern = work ? k_sampled_q<true, 16> : k_sampled_q<false, 16>;
    }
    res = resident_blocks(kern, L);
    W = plan_units(p.sample_runs, 0, p.n_samples, tiles, split, res, grab);
    sa_status rc = fill_u32(grab, 8 * kGrabStride, 0u, st, err);
    if (rc != SA_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0, st, nodes, s.verts,
                       s.height, p.samples, p.n_samples, W, point_args(pts, s),
                       SampOut{counts, minutes, bits, longest, scale, 0}, work);
    SA_CHECK_LAUNCH("sampled kernel");
    return SA_OK;
}

sa_status run_spill(const DeviceScene &s, const DevicePath &p, const ViewEntry *views, int j0, const PointArgs &P,
                    float scale, int32_t *counts, float *minutes, double *minutes64, SpillQueue &q, hipStream_t st,
                    std::string &err)
{
    hipLaunchKernelGGL(has_blocks(s.n_b) ? k_spill<true> : k_spill<false>, dim3(kSpillBlocks), dim3(kThreads), 0, st, views, s.n_b, j0, s.voff, s.verts,
                       s.height, p.segs, P, scale, counts, minutes, minutes64, (const int4 *)q.entries,
                       q.counters, q.capacity);
    SA_CHECK_LAUNCH("accrual spill");
    return SA_OK;
}

sa_status fill_u32(void *p, int64_t n, uint32_t v, hipStream_t st, std::string &err)
{
    if (n <= 0) return SA_OK;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, (uint32_t *)p, n, v);
    SA_CHECK_LAUNCH("fill");
    return SA_OK;
}

sa_status launch_batched(const DeviceScene &s, const DevicePath &p, int32_t n_var, int32_t k, const int32_t *ids,
                         const float *h, const PointsView &pts, const int64_t *var_off, float scale, int32_t *counts,
                         float *minutes, const TileLaunch &L, uint32_t *grab, uint32_t *flag, Scratch &scr,
                         Scratch &views_scr, Scratch &piece_scr, hipStream_t st, std::string &err)
{
    if (n_var == 0 || pts.n == 0) return SA_OK;
    // every variant may end with a tile of its own
    int64_t tiles;
    if (!tile_count(pts.n / 64 * 64 + (int64_t)n_var * 64, tiles, err)) return SA_ERR_INVALID_ARG;
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    size_t need = 0;
    auto part = [&](size_t bytes) {
        const size_t at = need;
        need += up(bytes);
        return at;
    };
    const size_t h_at = part(sizeof(float) * (size_t)n_var * s.n_b);
    const size_t tops_at = part(sizeof(float) * (size_t)s.n_b);
    const size_t tile_at = part(sizeof(int64_t) * (n_var + 1));
    if (!reserve(scr, need, st)) {
        err = "no room for the variants' heights (under stream capture an eager call of the size comes first)";
        return SA_ERR_OOM;
    }
    // on few tiles, runs in pieces as launch_accrual's
    const auto kern = has_blocks(s.n_b) ? k_batched<true> : k_batched<false>;
    const int64_t res = resident_blocks(kern, L);
    const bool pieces = tiles < 2 * res * kWaves;
    const int64_t max_parts = pieces ? piece_parts(piece_scr, pts.n, st) : 1;
    char *base = (char *)scr.ptr;
    float *vh = (float *)(base + h_at), *tops = (float *)(base + tops_at);
    int64_t *tile_off = (int64_t *)(base + tile_at);
    hipLaunchKernelGGL(k_var_copy, dim3(1024), dim3(256), 0, st, (const float *)s.height, s.n_b, n_var, vh, tops, var_off,
                       tile_off);
    const int64_t edits = (int64_t)n_var * k;
    if (s.n_b > 0 && edits > 0)
        hipLaunchKernelGGL(k_var_heights, dim3((unsigned)((edits + 255) / 256)), dim3(256), 0, st, edits, k, ids, h,
                           (const int32_t *)s.rank, s.n_b, vh, (int32_t *)tops, flag);
    SA_CHECK_LAUNCH("variant set-up");
    const PointArgs P = point_args(pts, s);
    // segment ranges whose views fit the per-launch budget; outputs accumulate
    // across the launches
    const int64_t per = seg_views_cap(s, p, views_scr, st);
    for (int64_t j0 = 0; j0 < p.n_segs; j0 += per) {
        const int j1 = (int)std::min<int64_t>(j0 + per, p.n_segs);
        ViewEntry *views = nullptr;
        sa_status rc = build_seg_views(s, p.segs, tops, (int)j0, j1, views_scr, {nullptr, grab, 8 * kGrabStride}, st, views, err);
        if (rc != SA_OK) return rc;
        const Sched W = plan_units(p.seg_runs, (int)j0, j1, tiles, pieces ? Split::kRunPieces : Split::kUniqueBins, res, grab,
                                   max_parts);
        BinOut O{counts, minutes, nullptr, nullptr, nullptr, 0, 0, scale, 0};
        if (W.sub > 1) {
            const size_t cnt_bytes = (size_t)W.n_parts * (size_t)pts.n * sizeof(int32_t);
            O.pcnt = (int32_t *)piece_scr.ptr;
            O.pmin = (double *)((char *)piece_scr.ptr + ((cnt_bytes + 255) & ~(size_t)255));
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0, st,
                           roof_boxes(s), views, s.n_b, s.voff, s.verts, (const float *)vh,
                           p.segs, (int)j0, j1, W, P, O, var_off, (const int64_t *)tile_off, n_var, flag);
        SA_CHECK_LAUNCH("batched accrual");
        if (W.sub > 1) {
            add_pieces(W, (int)j0, p, pts.n, O, var_off, n_var, st);
            SA_CHECK_LAUNCH("batched piece sums");
        }
    }
    return SA_OK;
}

int64_t seg_views_cap(const DeviceScene &s, const DevicePath &p, Scratch &scr, hipStream_t st)
{
    const int64_t per_seg = std::max<int64_t>(view_bytes(s.n_b), 1);
    if (scr.fixed) return (int64_t)scr.bytes / per_seg;
    if (s.n_b == 0) return std::max(p.n_segs, 1);
    auto fit = [&](int64_t budget) { return std::max<int64_t>(1, std::min<int64_t>(budget / per_seg, p.n_segs)); };
    for (int64_t budget = kViewBytes; budget > kLeastViewBytes; budget /= 2)
        if (reserve_wish(scr, (size_t)(fit(budget) * per_seg), st)) return fit(budget);
    const int64_t held = (int64_t)scr.bytes / per_seg;
    return std::max<int64_t>(held, capturing(st) ? 1 : fit(kLeastViewBytes));
}

sa_status build_seg_views(const DeviceScene &s, const SegConst *segs, const float *tops, int j0, int j1, Scratch &scr,
                          const LaunchState &state, hipStream_t st, ViewEntry *&views, std::string &err)
{
    views = nullptr;
    if (s.n_b == 0 || j1 <= j0) {
        hipLaunchKernelGGL(k_clear_state, dim3(1), dim3(256), 0, st, state);
        SA_CHECK_LAUNCH("launch state");
        return SA_OK;
    }
    const size_t need = (size_t)(j1 - j0) * view_bytes(s.n_b);
    if (scr.bytes < need && scr.fixed) {
        err = "per-segment views need " + std::to_string(need) + " bytes, more than the fixed " +
              std::to_string(scr.bytes);
        return SA_ERR_CAPACITY;
    }
    if (!reserve(scr, need, st)) {
        err = "no room for the segment views (under stream capture an eager call of the size comes first)";
        return SA_ERR_OOM;
    }
    views = (ViewEntry *)scr.ptr;
    launch_views(s, tops, segs, j0, j1, views, state, st);
    SA_CHECK_LAUNCH("segment views");
    return SA_OK;
}

// Output mode of an accrual launch starting at segment j0: with `store`
// (no SA_FLAG_ADD, and every bin's segments one contiguous run) a bin is
// stored by the launch holding its first segment and added to by later
// ones, so the outputs need no clearing.
static BinOut bin_out(const DevicePath &p, int j0, bool store, int32_t *counts, float *minutes, double *minutes64,
                      float scale)
{
    const bool first = store && (j0 == 0 || p.seg_bin[j0 - 1] != p.seg_bin[j0]);
    return BinOut{counts, minutes, minutes64, nullptr, nullptr, first ? 1 : 0, store ? 1 : 0, scale, 0};
}

sa_status launch_accrual(const DeviceScene &s, const DevicePath &p, const PointsView &pts, float scale,
                         int32_t *counts, float *minutes, double *minutes64, float *longest, uint64_t *work,
                         bool store, const TileLaunch &L, SpillQueue &q, Scratch &scr, Scratch &piece_scr,
                         hipStream_t st, std::string &err)
{
    const int32_t seg_per_launch = L.segments_per_launch;
    if (pts.n == 0) return SA_OK;
    int64_t tiles;
    if (!tile_count(pts.n, tiles, err)) return SA_ERR_INVALID_ARG;
    const PointArgs P = point_args(pts, s);
    // Long spans run as several launches over consecutive segment ranges,
    // each of at most kSpillWork point-segments and covering at most
    // kViewBytes of views (built just before it);
    // outputs are accumulated, so the split is invisible in the results.
    const int64_t cap = seg_views_cap(s, p, scr, st);
    if (s.n_b > 0 && p.n_segs > 0 && cap < 1) {
        err = "one segment's view (" + std::to_string(view_bytes(s.n_b)) +
              " bytes) exceed the fixed scratch (" + std::to_string(scr.bytes) + " bytes)";
        return SA_ERR_CAPACITY;
    }
    int64_t per = std::min(std::max<int64_t>(1, kSpillWork / (64 * tiles)), std::max<int64_t>(cap, 1));
    if (seg_per_launch > 0) per = std::min<int64_t>(per, seg_per_launch);
    if (longest) {
        // whole days per launch, so a run never spans two launches (one
        // day per launch at least, whatever its views take)
        const int D = (int)p.day_seg_off.size() - 1;
        if (scr.fixed && s.n_b > 0)
            for (int d = 0; d < D; ++d)
                if (p.day_seg_off[d + 1] - p.day_seg_off[d] > cap) {
                    err = "one day's views (" + std::to_string(p.day_seg_off[d + 1] - p.day_seg_off[d]) +
                          " segments) exceed the fixed scratch (" + std::to_string(cap) + " segments fit)";
                    return SA_ERR_CAPACITY;
                }
        for (int d0 = 0; d0 < D;) {
            int d1 = d0 + 1;
            while (d1 < D && p.day_seg_off[d1 + 1] - p.day_seg_off[d0] <= per) ++d1;
            const int j0 = p.day_seg_off[d0], j1 = p.day_seg_off[d1];
            ViewEntry *views;
            sa_status rc = build_seg_views(s, p.segs, s.height, j0, j1, scr, {nullptr, q.grab, 8 * kGrabStride}, st, views, err);
            if (rc != SA_OK) return rc;
            const auto kern = has_blocks(s.n_b) ? k_accrual_runs<true> : k_accrual_runs<false>;
            const int64_t res = resident_blocks(kern, L);
            const Sched W = plan_units(p.seg_runs, j0, j1, tiles, Split::kUniqueBins, res, q.grab);
            hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0,
                               st, roof_boxes(s), views, s.n_b, s.voff, s.verts, s.height, p.segs, j0, j1, W, P,
                               bin_out(p, j0, store, counts, minutes, minutes64, scale), longest, q.counters + 2);
            SA_CHECK_LAUNCH("accrual kernel (continuous shadow)");
            d0 = d1;
        }
        return SA_OK;
    }
    // (scenes of several blocks at eight waves per SIMD alone)
    auto kern = work ? k_accrual<true, 8, false> : k_accrual<false, 8, false>;
    if (L.waves_per_simd == 6) kern = work ? k_accrual<true, 6, false> : k_accrual<false, 6, false>;
    if (L.waves_per_simd == 7) kern = work ? k_accrual<true, 7, false> : k_accrual<false, 7, false>;
    if (has_blocks(s.n_b)) kern = work ? k_accrual<true, 8, true> : k_accrual<false, 8, true>;
    const int64_t res = resident_blocks(kern, L);
    // Too few tiles to give every resident wave several (tile, bin) units:
    // each bin's run is then cut into pieces, held as per-piece sums in
    // piece_scr ([part][n] counts, then, 256-byte aligned, FP64 minutes) and
    // added up in order by a second kernel, so the results stay deterministic.
    // Without room for the sums, whole runs.
    const bool pieces = tiles < 2 * res * kWaves;
    const int64_t max_parts = pieces ? piece_parts(piece_scr, pts.n, st) : 1;
    for (int64_t j0 = 0; j0 < p.n_segs; j0 += per) {
        const int j1 = (int)std::min<int64_t>(j0 + per, p.n_segs);
        ViewEntry *views;
        sa_status rc = build_seg_views(s, p.segs, s.height, (int)j0, j1, scr, {q.counters, q.grab, 8 * kGrabStride},
                                       st, views, err);
        if (rc != SA_OK) return rc;
        SpillArgs S{q.entries, q.counters, q.capacity};
        const Sched W = plan_units(p.seg_runs, (int)j0, j1, tiles, pieces ? Split::kRunPieces : Split::kUniqueBins,
                                   res, q.grab, max_parts);
        BinOut O = bin_out(p, (int)j0, store, counts, minutes, minutes64, scale);
        if (W.sub > 1) {
            const size_t cnt_bytes = (size_t)W.n_parts * (size_t)pts.n * sizeof(int32_t);
            O.pcnt = (int32_t *)piece_scr.ptr;
            O.pmin = (double *)((char *)piece_scr.ptr + ((cnt_bytes + 255) & ~(size_t)255));
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0, st, roof_boxes(s), views, s.n_b,
                           s.voff, s.verts, s.height, p.segs, (int)j0, j1, W, P, O, S, work);
        SA_CHECK_LAUNCH("accrual kernel");
        if (W.sub > 1) {
            add_pieces(W, (int)j0, p, pts.n, O, nullptr, 0, st);
            SA_CHECK_LAUNCH("accrual piece sums");
        }
        rc = run_spill(s, p, views, (int)j0, P, scale, counts, minutes, minutes64, q, st, err);
        if (rc != SA_OK) return rc;
    }
    return SA_OK;
}

sa_status launch_contribution(const DeviceScene &s, const DevicePath &p, const PointsView &pts, const float *weight,
                              double *contrib, const TileLaunch &L, uint32_t *grab, Scratch &scr, hipStream_t st,
                              std::string &err)
{
    if (pts.n == 0 || s.n_b == 0) return SA_OK;
    int64_t tiles;
    if (!tile_count(pts.n, tiles, err)) return SA_ERR_INVALID_ARG;
    const PointArgs P = point_args(pts, s);
    // long spans: several launches over consecutive segment ranges
    const int64_t per =
        std::min(std::max<int64_t>(1, kChunkWork / std::max<int64_t>(pts.n, 1)), seg_views_cap(s, p, scr, st));
    for (int64_t j0 = 0; j0 < p.n_segs; j0 += per) {
        const int j1 = (int)std::min<int64_t>(j0 + per, p.n_segs);
        ViewEntry *views;
        sa_status rc = build_seg_views(s, p.segs_by_reach, s.height, (int)j0, j1, scr, {nullptr, grab, 8 * kGrabStride}, st,
                                       views, err);
        if (rc != SA_OK) return rc;
        // The sums are atomic: on few tiles the units are chunks of segments.
        // No lane retires here, so a walk is as long as the sun is low: with the
        // longest first, dealt out in turn, the parts are alike and none of the
        // long ones is left for the end (20,000 points: 242 -> 200 us on 4,000
        // prisms, 475 -> 409 on 15,000; 250,000 on 15,000: 1.82 -> 1.61 ms).  The
        // accrual form retires soonest under the lowest sun and gains nothing
        // from this order (60,000 points on 300 prisms: 133 -> 162 us).
        const auto kern = has_blocks(s.n_b) ? k_contrib<true> : k_contrib<false>;
        const int64_t res = resident_blocks(kern, L);
        const Split split = tiles < 2 * res * kWaves ? Split::kChunks : Split::kBinRuns;
        const Sched W = plan_units(p.seg_runs, (int)j0, j1, tiles, split, res, grab);
        hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0, st, views,
                           s.n_b, s.voff, s.verts, s.height, p.segs_by_reach, (int)j0, j1, W, P, weight,
                           (const int32_t *)s.order, contrib);
        SA_CHECK_LAUNCH("contribution kernel");
    }
    return SA_OK;
}

}  // namespace sa
