// The sampled form by fans of instants: one walk of the scene serves all
// the rays from a point toward up to 16 consecutive instants of a day.
//
// Between neighbouring instants the sun hardly moves, so a point's rays
// toward a chunk of instants fill a narrow fan, and the prisms they can meet
// are those the fan meets.  A wave takes 64 points and one chunk, walks the
// chunk's view (the accrual form's walk, against a fan that holds every ray
// of the chunk), and at a leaf tests
// the prism against the chunk's rays one by one, with the arithmetic of
// ray_prism.  A ray is shadowed if any prism blocks it, whatever the order of
// the walk, so the predicate per (point, instant) is the packet kernels' own.
// Each lane keeps its point's instants as a bit mask and retires when all
// are shadowed.
//
// Two launches per range of chunks and points: k_sampled_fan stores a mask
// word per (chunk, point), every (tile, chunk) on its own, so small point
// sets fill the device too; k_sampled_sum reads a point's words in time order
// into counts, minutes and runs, and k_sampled_bits shifts them into the
// output's bit vectors.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "sa_internal.h"
#include "traverse.h"
#include "unit_sched.h"
#include "views.h"

namespace sa {
namespace {
using namespace dev;

constexpr int kThreads = kSchedThreads;
constexpr int kWaves = kSchedWaves;
constexpr int64_t kViewBytes = 256ll << 20;  // views per launch
constexpr int64_t kMaskBytes = 256ll << 20;  // mask words per launch

typedef __attribute__((address_space(4))) const FanChunk cChunk;
typedef __attribute__((address_space(4))) const FanDirs cDirs;

// Lane kLane of the 16-lane row of r, in every lane of the row.
template <int kLane>
__device__ __forceinline__ float row_bcast(float r)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(r), 0x150 + kLane, 0xF, 0xF, true));
}

// Eight instants (lanes kAt .. kAt + 7 of the row) past two edges on the same
// side: d[k] = min (or max) of d[k], na ra[k] and nb rb[k].  The products
// take their reciprocal from the row by DPP, so the broadcast costs no
// instruction.  One asm block, in place: left to the compiler, the arrays are
// copied between registers at every branch and spill.  The block waits out
// the two states a DPP operand needs after it is written.
#define SA_RAY(K, AT, OP)                                                                    \
    "v_mul_f32_dpp %[t], %[ra], %[na] row_newbcast:" AT " row_mask:0xf bank_mask:0xf\n"      \
    "v_mul_f32_dpp %[u], %[rb], %[nb] row_newbcast:" AT " row_mask:0xf bank_mask:0xf\n"      \
    OP " %[d" K "], %[d" K "], %[t], %[u]\n"
#define SA_RAYS(D, A0, A1, A2, A3, A4, A5, A6, A7, OP)                                       \
    do {                                                                                     \
        float t_, u_;                                                                        \
        asm("s_nop 1\n" SA_RAY("0", A0, OP) SA_RAY("1", A1, OP) SA_RAY("2", A2, OP)          \
                SA_RAY("3", A3, OP) SA_RAY("4", A4, OP) SA_RAY("5", A5, OP) SA_RAY("6", A6, OP) \
                    SA_RAY("7", A7, OP)                                                      \
            : [d0] "+v"((D)[0]), [d1] "+v"((D)[1]), [d2] "+v"((D)[2]), [d3] "+v"((D)[3]),    \
              [d4] "+v"((D)[4]), [d5] "+v"((D)[5]), [d6] "+v"((D)[6]), [d7] "+v"((D)[7]),    \
              [t] "=&v"(t_), [u] "=&v"(u_)                                                   \
            : [ra] "v"(a.r), [na] "v"(a.num), [rb] "v"(b.r), [nb] "v"(b.num));               \
    } while (0)

struct Edge {
    float num, r;      // the point's distance to it, the reciprocal of the lane's instant
};

__device__ __forceinline__ void rays_out(float *s_out, const Edge &a, const Edge &b)
{
    SA_RAYS(s_out, "0", "1", "2", "3", "4", "5", "6", "7", "v_min3_f32");
    SA_RAYS(s_out + 8, "8", "9", "10", "11", "12", "13", "14", "15", "v_min3_f32");
}

__device__ __forceinline__ void rays_in(float *s_in, const Edge &a, const Edge &b)
{
    SA_RAYS(s_in, "0", "1", "2", "3", "4", "5", "6", "7", "v_max3_f32");
    SA_RAYS(s_in + 8, "8", "9", "10", "11", "12", "13", "14", "15", "v_max3_f32");
}
#undef SA_RAYS
#undef SA_RAY

// bits = 2 bits + (this lane's bit of m): an add with carry.
__device__ __forceinline__ uint32_t push_bit(uint32_t bits, uint64_t m)
{
    asm("v_addc_co_u32_e64 %0, vcc, %0, %0, %1" : "+v"(bits) : "s"(m) : "vcc");
    return bits;
}

struct Dz16 {
    float v[16];
};
typedef __attribute__((address_space(4))) const Dz16 cDz16;

// Rays toward the chunk's 16 instants against a prism: bit k of the result
// is instant k.  Lane l holds the horizontal direction (dx, dy) of instant
// l mod 16, dz all of them.  Per footprint edge n . (x - v) <= 0 the rays'
// crossings are num / den with num the point's (a lane's) and den the
// instant's: a lane forms its instant's reciprocal, the 16 products take it
// from the row.  The side of an edge (den > 0: the ray leaves through it) is
// the same for all 16 instants but for edges nearly parallel to the light, so
// the edges are sorted by side into scalar masks first, and two of a side cost
// two multiplies and one three-way min or max per ray (single edges: 7.0 ms
// against 5.8 on the scene below).  Values and comparisons are ray_prism's.
template <int... K>
__device__ __forceinline__ uint32_t chunk_rays(std::integer_sequence<int, K...>, cfloat4 *verts, int voff, int m, float H,
                                               float px, float py, float pz, float dx, float dy, const Dz16 &dz)
{
    float s_in[16], s_out[16];
    ((s_in[K] = 0.f, s_out[K] = INFINITY), ...);
    for (int e0 = 0; e0 < m; e0 += 64) {
        const int ne = min(m - e0, 64);
        // the edges by side: masks of those all 16 rays leave or enter through
        uint64_t out = 0, in = 0;
        for (int e = 0; e < ne; ++e) {
            const float4 v = ld(verts + voff + e0 + e);
            const float den = fmaf(v.z, dx, v.w * dy);
            out |= (uint64_t)(gt_mask(den, 0.f) == ~0ull) << e;
            in |= (uint64_t)(lt_mask(den, 0.f) == ~0ull) << e;
        }
        uint64_t rest = (ne < 64 ? (1ull << ne) - 1ull : ~0ull) & ~(out | in);
        auto next = [&](uint64_t &set) {
            const int e = e0 + (int)__builtin_ctzll(set);
            set &= set - 1;
            const float4 v = ld(verts + voff + e);
            const float wx = v.x - px, wy = v.y - py;
            return Edge{fmaf(v.z, wx, v.w * wy), __builtin_amdgcn_rcpf(fmaf(v.z, dx, v.w * dy))};
        };
        // an odd last one pairs with itself (min and max are idempotent)
        while (out) {
            const Edge a = next(out);
            Edge b = a;
            if (out) b = next(out);
            rays_out(s_out, a, b);
        }
        while (in) {
            const Edge a = next(in);
            Edge b = a;
            if (in) b = next(in);
            rays_in(s_in, a, b);
        }
        while (rest) {
            const float4 v = ld(verts + voff + e0 + (int)__builtin_ctzll(rest));
            const float den = fmaf(v.z, dx, v.w * dy);
            const uint32_t o = (uint32_t)gt_mask(den, 0.f), i = (uint32_t)lt_mask(den, 0.f);
            const Edge g = next(rest);
            auto one = [&](float s, uint32_t ok, uint32_t ik, float &si, float &so) {
                so = ok ? fminf(so, s) : so;
                si = ik ? fmaxf(si, s) : si;
                so = (!(ok | ik) && g.num < 0.f) ? -INFINITY : so;  // parallel and outside
            };
            (one(g.num * row_bcast<K>(g.r), o >> K & 1u, i >> K & 1u, s_in[K], s_out[K]), ...);
        }
    }
    uint32_t hits = 0;
    ((hits = push_bit(hits, ge_mask(s_out[15 - K], s_in[15 - K]) &
                                le_mask(fmaf(s_in[15 - K], dz.v[15 - K], pz), H))),
     ...);
    return hits;
}

// Back-facing instants of a facade point: bit k is instant k.
template <int... K>
__device__ __forceinline__ uint32_t chunk_back(std::integer_sequence<int, K...>, float nx, float ny, const Dz16 &dx,
                                               const Dz16 &dy)
{
    uint32_t back = 0;
    ((back = push_bit(back, le_mask(fmaf(nx, dx.v[15 - K], ny * dy.v[15 - K]), 0.f))), ...);
    return back;
}

// Bound by VALU issue (94 % of it on the block scene): 1M points of the
// 20,000-prism scene over three days (2.16e9 rays) take 3.9 ms against 26.2 ms
// for the packets, with 3.8e6 leaf visits of 400 live rays each.  Over the binary
// hierarchy it was 5.0 ms (4.8e7 node fetches); there chunks of 32 instants walked
// less (2.8e7 fetches) but tested more rays a leaf (7.4 against 7.0 ms, both
// before the edges were paired), and 6, 7 and 8 waves per SIMD took 5.8, 5.5 and
// 5.4 ms, 161, 173 and 184 us on 20,000 points and 400 prisms, where a wave's own
// latency counts and the scalar registers spilled at 7 and 8 are felt.
template <bool kCount, bool kBlocks>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(7))) void k_sampled_fan(
    const ViewEntry *views_g, int n_b, const int32_t *voff_g, const float4 *verts_g, const float *height_g,
    const FanChunk *chunks_g, const FanDirs *dirs_g, int c0, int c1, Sched W, PointArgs P, uint16_t *masks,
    uint64_t *work)
{
    constexpr std::make_integer_sequence<int, 16> kSeq{};
    Work wk{0, 0, 0, 0, 0, 0, 0};
    cfloat4 *verts = (cfloat4 *)verts_g;
    cfloat *height = (cfloat *)height_g;
    cChunk *chunks = (cChunk *)chunks_g;
    __shared__ int s_W[sizeof(Sched) / 4];
    __shared__ int s_P[sizeof(PointArgs) / 4];
    __shared__ uint16_t *s_masks;
    if (tid() == 0) {
        lds_park((lds_int *)s_W, W);
        lds_park((lds_int *)s_P, P);
        s_masks = masks;
    }
    __syncthreads();
    __shared__ TileFan s_tile[kWaves];
    TileFan *tile = &s_tile[tid() >> 6];
    const int lane = tid() & 63;
    int kx = 0;
    Unit un;
    while (next_unit((lds_int *)s_W, c0, c1, kx, un)) {
        const int ca = uniform(un.a), cb = uniform(un.b), step = uniform(un.step);
        const PointArgs Pd = lds_uniform<PointArgs>((lds_int *)s_P);
        const int64_t n = Pd.n;
        const int64_t i = (int64_t)un.tile * 64 + lane;
        const bool valid = i < n;
        const LanePoint q = load_point(Pd, i, valid);
        const bool facades = ballot(q.own >= 0) != 0;
        for (int c = ca; c < cb; c += step) {
            const FanChunk ch = ld(chunks + c);
            cDirs *dd = (cDirs *)(dirs_g + c);
            const uint32_t all = (1u << ch.n) - 1u;
            uint32_t pend = valid ? all : 0u;  // instants not yet found shadowed
            if (facades) {
                const uint32_t back = chunk_back(kSeq, q.nx, q.ny, ld((cDz16 *)dd->dx), ld((cDz16 *)dd->dy));
                if (q.own >= 0) pend &= ~back;
            }
            if constexpr (kCount) wk.units += valid ? (uint32_t)ch.n : 0u;
            if (views_g != nullptr) {
                const float dx = dirs_g[c].dx[lane & 15], dy = dirs_g[c].dy[lane & 15];
                auto leaf = [&](int prim, int voff, int m, uint64_t want) -> uint64_t {
                    const uint64_t gm = want & ballot(prim != q.own);
                    if (!gm) return 0;
                    if constexpr (kCount) {
                        const uint32_t rays = lane_in(gm) ? (uint32_t)__builtin_popcount(pend) : 0u;
                        wk.prism += rays;
                        wk.edges += rays * (uint32_t)m;
                        wk.leaves += first_active_lane() ? 1u : 0u;
                    }
                    const uint32_t hits = chunk_rays(kSeq, verts, voff, m, ld(height + prim), q.px, q.py, q.pz, dx, dy,
                                                     ld((cDz16 *)dd->dz));
                    pend &= lane_in(gm) ? ~hits : ~0u;
                    return gm & ballot(pend == 0u);
                };
                const SegFan ft(fan_geom(ch), q.px, q.py, q.pz);
                walk_view<kCount, kBlocks>(views_g + (int64_t)(c - c0) * view_shape<kBlocks>(n_b).all, n_b, (cint *)voff_g, tile,
                                  ballot(pend != 0u), ft, leaf, wk);
            }
            if (valid) s_masks[(int64_t)(c - c0) * n + i] = (uint16_t)(all & ~pend);
        }
    }
    if constexpr (kCount) flush_work(wk, work);
}

struct FanSums {
    int32_t *counts;
    float *minutes;
    float *longest;
    int64_t n;      // row stride of the outputs
    float scale;
    int32_t store;  // a bin whose first chunk lies in the launch is stored, not added to
};

// A point's masks of chunks [ca, cb) in time order: counts, minutes and runs
// per bin, a run reset at each day's first instant.  With parts (part_start
// given) the launch's y index takes one bin run each.  Chunks whose instants
// weigh the same (all but a day's first and last) add their weight times the
// number of shadowed instants.
// Masks are asked for 32 at a time (a round trip to words that other XCDs have
// just written takes 2 us): 20,000 points, 46 chunks, 25 us one by one, 13 so.
constexpr int kMasksInFlight = 32;

typedef __attribute__((address_space(4))) const ChunkSum cSum;

__global__ __launch_bounds__(64) void k_sampled_sum(const uint16_t *__restrict__ masks, int64_t n, int64_t i0,
                                                    const ChunkSum *__restrict__ sums_g,
                                                    const SampleConst *__restrict__ samples_g, int c0, int c1,
                                                    const int32_t *__restrict__ part_start, FanSums O)
{
    __shared__ uint16_t s_w[kMasksInFlight][64];  // a column per thread
    const int64_t t = (int64_t)wg_id() * 64 + tid();
    if (t >= n) return;
    cSum *sums = (cSum *)sums_g;
    cSample *samples = (cSample *)samples_g;
    int ca = c0, cb = c1;
    if (part_start) {
        ca = max(ld((cint *)part_start + wg_id_y()), c0);
        cb = min(ld((cint *)part_start + wg_id_y() + 1), c1);
    }
    int cnt = 0, bin = ld(sums + ca).bin;
    float mins = 0.f, run = 0.f, best = 0.f;
    // the bin's run starts at chunk ca, in this launch or before it
    bool fresh = O.store && (ca == 0 || ld(sums + ca - 1).bin != bin);
    auto put = [&]() {
        const int64_t o = (int64_t)bin * O.n + i0 + t;
        if (O.counts) O.counts[o] = (fresh ? 0 : O.counts[o]) + cnt;
        if (O.minutes) O.minutes[o] = (fresh ? 0.f : O.minutes[o]) + mins * O.scale;
        if (O.longest) O.longest[o] = fmaxf(fresh ? 0.f : O.longest[o], best * O.scale);
    };
    for (int cc = ca; cc < cb; cc += kMasksInFlight) {
        uint16_t got[kMasksInFlight];
#pragma unroll
        for (int u = 0; u < kMasksInFlight; ++u) got[u] = masks[(int64_t)(min(cc + u, cb - 1) - c0) * n + t];
#pragma unroll
        for (int u = 0; u < kMasksInFlight; ++u) s_w[u][tid()] = got[u];
        for (int u = 0; u < min(kMasksInFlight, cb - cc); ++u) {
            const ChunkSum ch = ld(sums + cc + u);
            const uint32_t w = s_w[u][tid()];
            if (ch.bin != bin) {
                put();
                cnt = 0;
                mins = best = 0.f;
                bin = ch.bin;
                fresh = O.store != 0;
            }
            if (ch.n_flags & kSumDayStart) run = 0.f;
            const int on = __builtin_popcount(w);
            cnt += on;
            if ((ch.n_flags & kSumEven) && !O.longest) {
                mins = fmaf((float)on, ch.weight, mins);
                continue;
            }
            for (int k = 0; k < (ch.n_flags & 0xff); ++k) {
                const float wt = ld(samples + ch.first + k).w;
                const bool sh = (w >> k) & 1u;
                mins += sh ? wt : 0.f;
                run = sh ? run + wt : 0.f;
                best = fmaxf(best, run);
            }
        }
    }
    put();
}

// The launch's part of the output words [w0, w1): a word's chunks (two where
// a day ends inside it) shifted into place; a word begun by an earlier launch
// is added to.
__global__ __launch_bounds__(kThreads) void k_sampled_bits(const uint16_t *__restrict__ masks, int64_t n, int64_t i0,
                                                           const FanChunk *__restrict__ chunks, int c0, int c1, int w0,
                                                           int64_t n_out, uint32_t *__restrict__ bits)
{
    const int64_t t = (int64_t)wg_id() * kThreads + tid();
    const int w = w0 + (int)wg_id_y();
    if (t >= n) return;
    // the word's chunks follow one another; the first one by bisection
    int lo = c0, hi = c1 - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((chunks[mid].first >> 5) < w) lo = mid + 1;
        else hi = mid;
    }
    uint32_t v = 0;
    const bool begun = (chunks[lo].first & 31) != 0;
    for (int c = lo; c < c1 && (chunks[c].first >> 5) == w; ++c)
        v |= (uint32_t)masks[(int64_t)(c - c0) * n + t] << (chunks[c].first & 31);
    const int64_t o = (int64_t)w * n_out + i0 + t;
    bits[o] = begun ? (bits[o] | v) : v;
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

sa_status launch_sampled_fan(const DeviceScene &s, const DevicePath &p, const PointsView &pts, float scale,
                             int32_t *counts, float *minutes, uint32_t *bits, float *longest, uint64_t *work, bool store,
                             const TileLaunch &L, uint32_t *grab, Scratch &views_scr, Scratch &mask_scr, bool &taken,
                             hipStream_t st, std::string &err)
{
    taken = false;
    if (pts.n == 0 || p.n_chunks == 0) {
        taken = true;
        return SA_OK;
    }
    // chunks per launch: their views fit the budget, and so do the words of as
    // many points as fill the device; whole days where runs of shadow must not
    // be cut
    const int64_t view = s.n_b > 0 ? view_bytes(s.n_b) : 0;
    const int64_t least = std::min<int64_t>((pts.n + 63) / 64 * 64, 1 << 14);
    int64_t per = kMaskBytes / (2 * least);
    if (view > 0) per = std::max<int64_t>(1, std::min(per, kViewBytes / view));
    std::vector<int> cut{0};
    for (int c = 1; c < p.n_chunks; ++c) {
        const bool may = !longest || p.chunk_day_start[c];
        // the next place a launch may end: here, if what follows up to the
        // next one would not fit
        if (!may) continue;
        int next = c + 1;
        while (longest && next < p.n_chunks && !p.chunk_day_start[next]) ++next;
        if (next - cut.back() > per) cut.push_back(c);
    }
    cut.push_back(p.n_chunks);
    int64_t most = 0;
    for (size_t k = 0; k + 1 < cut.size(); ++k) most = std::max<int64_t>(most, cut[k + 1] - cut[k]);
    // points per launch: their words fit the budget
    const int64_t fit = std::max<int64_t>(kMaskBytes / (most * 2) / 64 * 64, 64);
    const int64_t ranges = (pts.n + fit - 1) / fit;  // of equal length: no short last one
    const int64_t range = ((pts.n + ranges - 1) / ranges + 63) / 64 * 64;
    // no room: the caller's other kernels need none
    const size_t view_need = (size_t)(most * view), mask_need = (size_t)(most * range * 2);
    if (hopeless(views_scr, view_need) || !reserve_wish(mask_scr, mask_need, st)) return SA_OK;
    if (!reserve(views_scr, view_need, st)) {
        release(mask_scr, st);
        return SA_OK;
    }
    taken = true;
    uint16_t *masks = (uint16_t *)mask_scr.ptr;
    auto kern = work ? k_sampled_fan<true, false> : k_sampled_fan<false, false>;
    if (has_blocks(s.n_b)) kern = work ? k_sampled_fan<true, true> : k_sampled_fan<false, true>;
    const int64_t res = resident_blocks(kern, L);
    const auto &rs = p.chunk_runs.start;
    for (size_t k = 0; k + 1 < cut.size(); ++k) {
        const int c0 = cut[k], c1 = cut[k + 1];
        ViewEntry *views = nullptr;
        if (view > 0) {
            views = (ViewEntry *)views_scr.ptr;
            launch_views(s, s.height, (const FanChunk *)p.chunks, c0, c1, views,
                         LaunchState{nullptr, grab, 8 * kGrabStride}, st);
            SA_CHECK_LAUNCH("fan views");
        }
        // bin runs of the launch: summed by a thread each where no bin has two
        const int r0 = (int)(std::upper_bound(rs.begin(), rs.end(), c0) - rs.begin()) - 1;
        const int r1 = (int)(std::upper_bound(rs.begin(), rs.end(), c1 - 1) - rs.begin());
        const bool parts = p.chunk_bins_unique && r1 - r0 > 1 && r1 - r0 < 65536;
        for (int64_t i0 = 0; i0 < pts.n; i0 += range) {
            const int64_t n = std::min(range, pts.n - i0);
            const PointArgs P{n, pts.x + i0, pts.y + i0, pts.z + i0, pts.nx ? pts.nx + i0 : nullptr,
                              pts.ny ? pts.ny + i0 : nullptr, pts.owner ? pts.owner + i0 : nullptr, s.rank, s.n_b};
            const Sched W = plan_units(p.chunk_runs, c0, c1, (n + 63) / 64, Split::kChunks, res, grab);
            if (W.grab && (i0 > 0 || !views)) {  // later ranges: the views' kernel cleared the first's
                sa_status rc = fill_u32(grab, 8 * kGrabStride, 0u, st, err);
                if (rc != SA_OK) return rc;
            }
            hipLaunchKernelGGL(kern, dim3((unsigned)unit_blocks(res, W)), dim3(kThreads), 0, st, (const ViewEntry *)views,
                               s.n_b, s.voff, s.verts, s.height, (const FanChunk *)p.chunks,
                               (const FanDirs *)p.chunk_dirs, c0, c1, W, P, masks, work);
            SA_CHECK_LAUNCH("sampled fan kernel");
            const unsigned blocks = (unsigned)((n + kThreads - 1) / kThreads);
            if (counts || minutes || longest) {
                hipLaunchKernelGGL(k_sampled_sum, dim3((unsigned)((n + 63) / 64), parts ? (unsigned)(r1 - r0) : 1u),
                                   dim3(64), 0, st, (const uint16_t *)masks, n, i0, (const ChunkSum *)p.chunk_sums,
                                   (const SampleConst *)p.samples, c0, c1,
                                   parts ? (const int32_t *)p.chunk_runs.dev + r0 : nullptr,
                                   FanSums{counts, minutes, longest, pts.n, scale, store ? 1 : 0});
                SA_CHECK_LAUNCH("sampled sums");
            }
            if (bits) {
                const int w0 = p.chunk_first[c0] >> 5, w1 = (p.chunk_first[c1 - 1] >> 5) + 1;
                for (int w = w0; w < w1; w += 32768)
                    hipLaunchKernelGGL(k_sampled_bits, dim3(blocks, (unsigned)std::min(32768, w1 - w)), dim3(kThreads),
                                       0, st, (const uint16_t *)masks, n, i0, (const FanChunk *)p.chunks, c0, c1, w,
                                       pts.n, bits);
                SA_CHECK_LAUNCH("sampled bit vectors");
            }
        }
    }
    return SA_OK;
}

}  // namespace sa
