// Internal types shared by the library's host and device sources.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "shadow_accrual.h"

namespace sa {

// The work-item index within its work-group and the work-group index, read
// straight from the registers the hardware fills at dispatch.  The
// runtime's own accessors (threadIdx, blockIdx) are calls into its device
// library in this build: that library keeps IEEE mode on and the kernels
// turn it off, so the calls are not inlined, and a call site makes the
// register allocator keep to the calling convention (the accrual kernel
// spilled two vector registers to scratch memory for it).
__device__ __forceinline__ unsigned tid() { return __builtin_amdgcn_workitem_id_x(); }
__device__ __forceinline__ unsigned wg_id() { return __builtin_amdgcn_workgroup_id_x(); }
__device__ __forceinline__ unsigned wg_id_y() { return __builtin_amdgcn_workgroup_id_y(); }
// Work-items per work-group and work-groups in the grid (x), from the
// dispatch packet.
__device__ __forceinline__ unsigned wg_size() { return __builtin_amdgcn_workgroup_size_x(); }
__device__ __forceinline__ unsigned n_wg() { return __builtin_amdgcn_grid_size_x() / __builtin_amdgcn_workgroup_size_x(); }

// One interior node of the binary hierarchy: the boxes of both children
// (footprint-plane box x0,y0,x1,y1 and the top z1; every box starts at
// z = 0 because every prism stands on the ground) and the child
// references: >= 0 an interior node, < 0 the leaf ~prim (prism index in
// hierarchy order).  For leaf children the vertex range of the footprint
// is stored beside the reference so a leaf costs no extra indirection.
// 64 bytes: one scalar 16-dword load brings a whole node into SGPRs.
struct alignas(64) Node {
    float lx0, ly0, lx1, ly1;
    float rx0, ry0, rx1, ry1;
    float lz1, rz1;
    int32_t left, right;
    int32_t l_voff, l_m, r_voff, r_m;
};
static_assert(sizeof(Node) == 64, "node is one 64-byte line");

// Per sample instant, read uniformly by every lane of a wave.
struct alignas(32) SampleConst {
    float dx, dy, dz, w;  // unit direction toward the sun, weight (minutes)
    float ix, iy, iz;     // 1 / direction (components kept away from zero)
    int32_t tag;          // output bin | kDayStart on the first instant of a day
};
constexpr int32_t kDayStart = 1 << 30;
constexpr int32_t kBinMask = kDayStart - 1;

// Per great-circle segment of the accrual form.  In the segment's plane
// the direction at angle phi from the first knot is
// cos(phi) e1 + sin(phi) e2, phi in [0, theta], reached at time
// t = ta + dt * phi / theta.  An xy offset w from a point maps to the
// point of the plane above/below it, whose in-plane coordinates times
// |nz| (n = e1 x e2) are (u, v) = M w, and whose height above the point
// times |nz| is u * e1z + v * e2z (the factor keeps M bounded for planes
// through the zenith; directions are unchanged by it).
struct alignas(64) SegConst {
    float m00, m01, m10, m11;    // M (scaled by |nz|)
    float e1z, e2z, theta, dt;   // clip normal (u,v)->z, angle, minutes
    float ta;                    // start, minutes after local midnight
    float cth, sth;              // (cos theta, sin theta): end direction in (u, v)
    float nz;                    // vertical part of the plane normal e1 x e2
    int32_t mult;                // segments this one stands for (direction graph; else 1)
    int32_t ns_all;              // their sample instants
    int32_t bin;
    int32_t day;
    float e1x, e1y, e2x, e2y;    // horizontal parts of e1, e2 (facade back-face term)
    float ua_x, ua_y, ub_x, ub_y;  // horizontal offset per metre of rise, at both knots
    float s0;                    // first sample instant in the segment, minutes after ta
    float wrate;                 // minutes per radian the measure is weighted by: rate, or for a
                                 // direction-graph edge its segments' total duration / theta
    int32_t ns;                  // sample instants attributed to the segment
    int32_t steep;               // plane within 5 degrees of vertical: in-plane extreme search
    float rate;                  // dt / theta: minutes per radian
    float inv_step;              // 1 / step
    float mdx, mdy;              // horizontal part of the direction at theta / 2 (visit order)
};
static_assert(sizeof(SegConst) == 128, "two lines");

// What a segment (or a chunk of instants) makes of a prism or of a group of
// them: the box terms of the fan test (the box edges shifted by the fan's
// per-metre reach: x1 - z1 umnx, x0 - z1 umxx, y1 - z1 umny, y0 - z1 umxy; the
// two wedge projections), of a group the least strict of its members'.  A
// fan's view of the scene is the entries of the blocks of 64 groups of groups,
// of the groups of 64 groups, of the groups of 32 prisms (of each where there
// are two or more), and of the prisms, group by group along a Hilbert curve;
// siblings (up to 64 blocks, a block's groups of groups, those' groups, a
// group's prisms) nearest along the fan's middle direction first.
struct alignas(32) ViewEntry {
    float c[6];
    int32_t ref;    // prism (hierarchy position), group, or block
    uint32_t vert;  // prism: first vertex and, above kLeafVertBits, their number (0: see its offsets)
};
static_assert(sizeof(ViewEntry) == 32, "two 16-byte loads a lane");
constexpr int kGroupBits = 5;  // prisms per group
constexpr int kSuperBits = 6;  // groups per group of groups: as many as a wave has lanes
constexpr int kBlockBits = 6;  // groups of groups per block: as many again
constexpr int kLeafVertBits = 27;
struct ViewShape {
    int32_t n_b, n1, n2, n3;      // prisms, groups, groups of groups, blocks
    uint32_t at2, at1, at0, all;  // entries before the groups of groups, the groups, the prisms, in all
};
// (kBlocks = false: of a scene known to have one block, at most 131,072 prisms.)
template <bool kBlocks = true>
constexpr ViewShape view_shape(int32_t n_b)
{
    const int32_t n1 = (int32_t)(((uint32_t)n_b + (1u << kGroupBits) - 1u) >> kGroupBits);
    const int32_t n2 = (n1 + (1 << kSuperBits) - 1) >> kSuperBits;
    const int32_t n3 = kBlocks ? (n2 + (1 << kBlockBits) - 1) >> kBlockBits : 1;
    const uint32_t at2 = n3 > 1 ? (uint32_t)n3 : 0u;
    const uint32_t at1 = at2 + (n2 > 1 ? (uint32_t)n2 : 0u);
    const uint32_t at0 = at1 + (n1 > 1 ? (uint32_t)n1 : 0u);
    return {n_b, n1, n2, n3, at2, at1, at0, at0 + (uint32_t)n_b};
}
inline bool has_blocks(int32_t n_b) { return view_shape(n_b).n3 > 1; }
inline int64_t view_bytes(int32_t n_b) { return (int64_t)view_shape(n_b).all * (int64_t)sizeof(ViewEntry); }

// A chunk of the sampled form: up to kFanInstants consecutive instants of one
// day (never across a multiple of it, so within a word of the bit vectors), whose
// rays from a point fill the fan f: the per-metre reach box of their
// horizontal offsets (umnx, umxx, umny, umxy) and the inward normals of its
// two edges (nax, nay, nbx, nby; zero where the directions spread too far to
// be bounded by two edges).
constexpr int kFanInstants = 16;
struct alignas(64) FanChunk {
    float f[8];
    float mdx, mdy;     // middle direction (visit order)
    int32_t first, n;   // its instants [first, first + n)
    int32_t pad[4];
};
static_assert(sizeof(FanChunk) == 64, "one line");

// What adding up a chunk's shadowed instants takes, four to a line.
struct alignas(16) ChunkSum {
    int32_t first;
    int32_t n_flags;  // instants | kSumDayStart: it holds its day's first instant | kSumEven: they weigh the same
    int32_t bin;
    float weight;     // of each instant, if even (minutes)
};
constexpr int32_t kSumDayStart = 1 << 8, kSumEven = 1 << 9;

// Their directions; entries past n repeat the last one.
struct alignas(64) FanDirs {
    float dx[kFanInstants], dy[kFanInstants], dz[kFanInstants];
};

struct DeviceScene {
    int32_t n_b = 0;
    int32_t n_vert = 0;
    int32_t n_nodes = 0;
    int32_t depth = 0;
    float bounds[4] = {0, 0, 0, 0};
    float max_h = 0;
    Node *nodes = nullptr;       // [n_nodes]
    float4 *verts = nullptr;     // [n_vert] x, y, edge normal (ey, -ex) in hierarchy order
    int32_t *voff = nullptr;     // [n_b + 1] hierarchy order
    float *height = nullptr;     // [n_b] hierarchy order
    int32_t *order = nullptr;    // [n_b] hierarchy position -> original id
    int32_t *rank = nullptr;     // [n_b] original id -> hierarchy position
    int32_t *parent = nullptr;   // [n_nodes + n_b] parent*2+side of interior nodes then leaves
    int32_t *flags = nullptr;    // [n_nodes] refit arrival counters
    float4 *pbox = nullptr;      // [n_b] prism footprint boxes, hierarchy order
    int32_t *vorder = nullptr;   // [n_b] views' order: hierarchy positions along a Hilbert curve
    float4 *gbox = nullptr;      // [n1 + n2 + n3] footprint boxes of the groups, groups of groups and blocks (ViewShape)
    int32_t *leaf_depth = nullptr;  // [n_b] nodes above each prism, hierarchy order
};

// A few heights by hierarchy position, passed to a kernel by value.
constexpr int kMaxEdits = 64;
struct HeightEdits {
    int32_t n;
    int32_t pos[kMaxEdits];
    float h[kMaxEdits];
};

// Raster shadow accrual map (Sec. 4) of one segment: the shadow plane
// (normal a, the segment's start direction) and its texel grid, float32,
// every coordinate relative to the box centre o.
struct SamGrid {
    float ax, ay, az;  // plane normal
    float ux, uy, uz;  // in-plane basis, u horizontal
    float vx, vy, vz;
    float c;           // plane: (x - o).a = c
    float u0, v0;      // grid corner in (u, v)
    float h, inv_h;    // texel edge and its inverse
    int32_t nu, nv;    // texels along u and v
    float ox, oy, oz;  // o, world coordinates
    float bias;        // depth margin of the shadow test (m)
    float dq, inv_dq;  // depth quantum of the map words (m) and its inverse
};

// One slice: an instant's direction on the great circle between the
// segment's knots, 1 / (d.a) (distance along the light per distance from
// the plane), and the instant's minutes.
struct SamSlice {
    float dx, dy, dz, inv_da;
    float w;
    int32_t pad[3];
};

struct SamSegHost {
    double a[3], b[3];  // knot directions
    double ta, tb;      // knot times (local minutes)
    int32_t first, ns;  // its sample instants
    int32_t bin;
};

// Maximal runs of consecutive items (segments or instants) with the same
// output bin: where each starts (then the item count) and its bin, on the
// host, and the starts on the device.
struct BinRuns {
    std::vector<int32_t> start, bin;
    int32_t *dev = nullptr;
};

struct DevicePath {
    int32_t n_days = 0, n_samples = 0, n_segs = 0, n_bins = 0;
    SampleConst *samples = nullptr;  // [n_samples]
    SamSlice *sam_slices = nullptr;  // [n_samples] raster slices (unmerged paths)
    SegConst *segs = nullptr;        // [n_segs]
    SegConst *segs_by_reach = nullptr;  // [n_segs] each bin run's by the sun's height, lowest first (contributions)
    int32_t words = 0;               // ceil(n_samples / 32)
    std::vector<int32_t> day_seg_off;  // host: first segment of each day, [n_days + 1]
    std::vector<int32_t> seg_bin;      // host: output bin of each segment
    bool bins_contiguous = false;      // host: every bin has segments, all in one run
    BinRuns seg_runs;                  // runs of equal bins over the segments
    BinRuns sample_runs;               // and over the instants
    int32_t n_chunks = 0;              // fans of instants of the sampled form
    FanChunk *chunks = nullptr;        // [n_chunks]
    FanDirs *chunk_dirs = nullptr;     // [n_chunks]
    ChunkSum *chunk_sums = nullptr;    // [n_chunks]
    BinRuns chunk_runs;                // runs of equal bins over the chunks
    bool chunk_bins_unique = false;    // host: no bin has two runs
    bool chunk_bins_all = false;       // host: and every bin has one
    std::vector<int32_t> chunk_first;  // host: each chunk's first instant
    std::vector<char> chunk_day_start;  // host: whether it is its day's first
    std::vector<double> bin_span;      // host: daylight minutes of each output bin
    bool merged = false;               // host: segments merged into direction-graph edges
    // host, for the raster form: each segment's knot directions, times, its
    // instants [first, first + ns) and bin; every instant's time and weight
    std::vector<SamSegHost> seg_host;
    std::vector<double> sample_t, sample_w;
};

// The queue of spilled point-segments: entries (first point, segment, points
// from that one on as 64 bits) of one point first, then of a tile's, of which a
// launch of kSpillWork point-segments cannot need more.  One in 1e4 point-segments spills
// on the block scenes, one in 77 among thin towers.
constexpr uint32_t kSpillSingles = 1u << 20;
constexpr int32_t kSpillCapacity = 1 << 23;
constexpr int64_t kSpillWork = 64ll * kSpillCapacity;

// Scratch owned by a context (grown on demand, freed with it), or a fixed
// buffer the library never grows or frees (fixed = true).
struct Scratch {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool fixed = false;
    uint32_t made = 0;           // allocations so far: a change means new contents
    size_t refused = SIZE_MAX;   // the least size that could not be had
};

// Is the stream being captured, or may it be (the runtime does not say)?
inline bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return cs != hipStreamCaptureStatusNone;
}

inline void release(Scratch &scr, hipStream_t st)
{
    (void)hipStreamSynchronize(st);  // queued kernels may still read it
    (void)hipFree(scr.ptr);
    scr.ptr = nullptr;
    scr.bytes = 0;
}

// Room for `need` bytes in scr: what it holds, where that is enough; else new
// memory, once the stream's work is done with the old.  Not of a fixed one, nor
// under stream capture, which neither the wait nor the allocation may be part
// of: false, and scr is as it was.  False with nothing in scr where the memory
// cannot be had.
inline bool reserve(Scratch &scr, size_t need, hipStream_t st)
{
    if (scr.bytes >= need) return true;
    if (scr.fixed || capturing(st)) return false;
    release(scr, st);
    if (hipMalloc(&scr.ptr, need) != hipSuccess) {
        (void)hipGetLastError();
        scr.ptr = nullptr;
        scr.refused = std::min(scr.refused, need);
        return false;
    }
    scr.bytes = need;
    ++scr.made;
    if (need >= scr.refused) scr.refused = SIZE_MAX;
    return true;
}

// The same for a size the caller can do without: one that was refused (or a
// larger one) is not asked for again, and what scr holds stays.
inline bool hopeless(const Scratch &scr, size_t need) { return need > scr.bytes && need >= scr.refused; }
inline bool reserve_wish(Scratch &scr, size_t need, hipStream_t st) { return !hopeless(scr, need) && reserve(scr, need, st); }

// Host-side builders implemented in the .hip sources.
sa_status scene_build(DeviceScene &s, hipStream_t st, int32_t n_b, const int32_t *voff,
                      const float *xy, const float *h, std::string &err);
sa_status scene_refit(DeviceScene &s, hipStream_t st, std::string &err);
// Heights h of the prisms at hierarchy positions pos (host arrays, no position
// twice) into the scene, with the tops above them; scr: staging of long edits.
sa_status scene_edit_heights(DeviceScene &s, int32_t n, const int32_t *pos, const float *h, Scratch &scr, hipStream_t st,
                             std::string &err);
// Heights from device arrays ids / h (original ids) into the scene, on the
// stream; an id out of range or a height that is not a positive finite
// number is skipped and raises bit 2 of *flag.
sa_status scene_set_heights_device(DeviceScene &s, int32_t n, const int32_t *ids, const float *h, uint32_t *flag,
                                   hipStream_t st, std::string &err);
void scene_free(DeviceScene &s);
sa_status sunpath_fill(const sa_site &site, const sa_timespan &span, sa_sunpath_buf &out,
                       std::string &err);

struct PointsView {
    int64_t n;
    const float *x, *y, *z, *nx, *ny;
    const int32_t *owner;
};

struct SpillQueue {
    int4 *entries = nullptr;       // [kSpillSingles + capacity]
    uint32_t *counters = nullptr;  // [0], [1] entries of one point and of a tile's, [2] overflow flag
    uint32_t *grab = nullptr;      // the accrual launch's work counters (eight, 128 B apart)
    int32_t capacity = 0;
};

// Device words a launch finds at zero (either may be null); n_counters <= 256.
struct LaunchState {
    uint32_t *queue_lengths;  // two
    uint32_t *counters;
    int32_t n_counters;
};

// Launch choices of the per-tile kernels: the most segments one accrual
// launch covers (0: as many as the view budget allows) and the blocks of
// the persistent launches (0: as many as the device holds at once, from
// the kernel's occupancy and the device's compute units) and the accrual
// kernel's occupancy variant.
struct TileLaunch {
    int32_t segments_per_launch;
    int64_t grid_blocks;
    int32_t n_cu;
    int32_t waves_per_simd;  // the accrual kernel's occupancy variant: 6, 7 or 8 (0: 8)
    int32_t sampled_instants;  // instants per packet of the sampled form: 1, 2, 4, 8 or 16 (0: fans of
                               // instants; of packets where those cannot be, 8)
};

sa_status launch_sampled(const DeviceScene &s, const DevicePath &p, const PointsView &pts,
                         float scale, int32_t *counts, float *minutes, uint32_t *bits, float *longest,
                         uint64_t *work, const TileLaunch &L, uint32_t *grab, hipStream_t st,
                         std::string &err);
// The sampled form by fans of instants, with views and mask words in
// views_scr and mask_scr (grown as needed, with the stream synchronised
// first).  taken = false, with nothing enqueued, where they cannot be had (a
// size refused once is not asked for again): launch_sampled gives the same
// results without scratch.  store: outputs need
// no clearing (no SA_FLAG_ADD and p.chunk_bins_all).
sa_status launch_sampled_fan(const DeviceScene &s, const DevicePath &p, const PointsView &pts, float scale,
                             int32_t *counts, float *minutes, uint32_t *bits, float *longest, uint64_t *work, bool store,
                             const TileLaunch &L, uint32_t *grab, Scratch &views_scr, Scratch &mask_scr, bool &taken,
                             hipStream_t st, std::string &err);
// store: outputs need no clearing (no SA_FLAG_ADD and p.bins_contiguous):
// each bin is stored by the launch holding its first segment.
// L: the launch choices (segments per launch, persistent grid size).
// piece_scr: per-piece sums when the tiles are too few to fill the device
// (whole runs where there is no room for them).
sa_status launch_accrual(const DeviceScene &s, const DevicePath &p, const PointsView &pts,
                         float scale, int32_t *counts, float *minutes, double *minutes64, float *longest,
                         uint64_t *work, bool store, const TileLaunch &L, SpillQueue &q, Scratch &scr,
                         Scratch &piece_scr, hipStream_t st, std::string &err);
// grad = (add ? grad : 0) + scale * d(sum dl * minutes)/dH, accumulated in
// FP64 in acc (grown to n_b doubles as needed).
sa_status launch_grad(const DeviceScene &s, const DevicePath &p, const PointsView &pts,
                      const float *dl, float scale, bool add, float *grad, const TileLaunch &L, SpillQueue &q,
                      Scratch &scr, Scratch &acc, hipStream_t st, std::string &err);
sa_status launch_region_sum(const float *v, int n_bins, int64_t n, const double *bin_w,
                            const int64_t *off, int32_t n_reg, const float *area, double *out,
                            Scratch &scr, hipStream_t st, std::string &err);
// The FP32 FMA lane-op rate the device sustains (a roofline measurement aid).
sa_status measure_valu_peak(int n_cu, float *sink, int64_t sink_floats, hipStream_t st, double &lane_ops_per_s,
                            std::string &err);
sa_status launch_contribution(const DeviceScene &s, const DevicePath &p, const PointsView &pts,
                              const float *weight, double *contrib, const TileLaunch &L, uint32_t *grab,
                              Scratch &scr, hipStream_t st, std::string &err);
// Views of segments [j0, j1) into scr (reserved; a fixed scr that is too small
// is a CAPACITY error), one after the other, and `state` cleared; views = nullptr for an empty scene.
// `tops`: the prisms' heights the views take (hierarchy order).
// seg_views_cap: segments whose views a launch takes: the per-launch budget,
// less where scr cannot be grown to it (of a fixed scr what fits, 0 if not even
// one does; under stream capture what fits, at least one).
sa_status build_seg_views(const DeviceScene &s, const SegConst *segs, const float *tops, int j0, int j1, Scratch &scr,
                          const LaunchState &state, hipStream_t st, ViewEntry *&views, std::string &err);
int64_t seg_views_cap(const DeviceScene &s, const DevicePath &p, Scratch &scr, hipStream_t st);
// Gross shadow by raster shadow accrual maps (Sec. 4) into counts/minutes
// [n_bins * n] (already cleared): per segment a map of slices x nu x nv
// 32-bit words (stamp, depth) in scr (grown as needed; max_texels caps one
// segment's map, with cap_both the two it may keep); stamp: the last segment stamp written into scr, kept by
// the caller with scr.
sa_status launch_sam(const DeviceScene &s, const DevicePath &p, const PointsView &pts, double texel,
                     double bias, const double box[6], int64_t max_texels, bool cap_both, float scale, int32_t *counts,
                     float *minutes, Scratch &scr, uint32_t &stamp, hipStream_t st, std::string &err);
sa_status launch_batched(const DeviceScene &s, const DevicePath &p, int32_t n_var, int32_t k,
                         const int32_t *ids, const float *h, const PointsView &pts,
                         const int64_t *var_off, float scale, int32_t *counts, float *minutes,
                         const TileLaunch &L, uint32_t *grab, uint32_t *flag, Scratch &scr, Scratch &views_scr,
                         Scratch &piece_scr, hipStream_t st, std::string &err);
// Graph-capturable fill of n 32-bit words.
sa_status fill_u32(void *p, int64_t n, uint32_t v, hipStream_t st, std::string &err);

}  // namespace sa
