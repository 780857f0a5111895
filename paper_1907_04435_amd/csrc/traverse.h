// Device-side building blocks shared by the traversal kernels.
//
// Traversal is wave-coherent: a wave of 64 lanes (64 neighbouring points,
// one sun instant or one path segment) walks the scene as one packet.
// Segments and fans of instants go by views of it (walk_view, below), roof
// tests by the boxes of the views' groups (roof_covered), single instants by
// the binary hierarchy.  There the node index is wave-uniform, so a node is
// fetched once per wave with a scalar load into SGPRs; each lane tests the two
// child boxes against its own ray; a child is entered when any still-live lane
// needs it.  The traversal stack is wave-uniform too: one 64-entry array per
// wave in LDS (every lane writes the same entry, pops are broadcast reads), so
// no per-lane stack and no scratch memory is needed.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "sa_internal.h"

namespace sa {
namespace dev {

constexpr int32_t kNone = INT_MIN;

typedef __attribute__((address_space(4))) const Node cNode;
typedef __attribute__((address_space(4))) const float4 cfloat4;
typedef __attribute__((address_space(4))) const float cfloat;
typedef __attribute__((address_space(4))) const SampleConst cSample;
typedef __attribute__((address_space(4))) const SegConst cSeg;

typedef __attribute__((address_space(4))) const int cint;

// Word-wise copy out of the constant address space: with a wave-uniform
// address this becomes one scalar load of the whole object.
template <class T>
__device__ __forceinline__ T ld(const __attribute__((address_space(4))) T *p)
{
    static_assert(sizeof(T) % 4 == 0, "word-sized objects");
    T r;
    int *d = (int *)&r;
    cint *s = (cint *)p;
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) d[i] = s[i];
    return r;
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Lane masks of float comparisons: one compare each, straight into a mask
// (no round trip through a per-lane boolean).
__device__ __forceinline__ uint64_t ge_mask(float a, float b) { return __builtin_amdgcn_fcmpf(a, b, 3); }
__device__ __forceinline__ uint64_t le_mask(float a, float b) { return __builtin_amdgcn_fcmpf(a, b, 5); }
__device__ __forceinline__ uint64_t lt_mask(float a, float b) { return __builtin_amdgcn_fcmpf(a, b, 4); }
__device__ __forceinline__ uint64_t gt_mask(float a, float b) { return __builtin_amdgcn_fcmpf(a, b, 2); }
__device__ __forceinline__ uint64_t to_mask(bool b) { return ballot(b); }
__device__ __forceinline__ uint64_t to_mask(uint64_t m) { return m; }

constexpr int kStackDepth = 64;

// Box padding of the hierarchy: absorbs the rounding of the slab test at
// large coordinates (boxes only decide what is tested, never a result).
__device__ __forceinline__ float pad_lo(float v) { return v - (1e-2f + fabsf(v) * 0x1p-20f); }
__device__ __forceinline__ float pad_hi(float v) { return v + (1e-2f + fabsf(v) * 0x1p-20f); }

// Work a lane's own traversal needed (instrumented instantiations only).
struct Work {
    uint32_t box, prism, edges, inserts, nodes, units, spills, leaves;
};

__device__ __forceinline__ bool first_active_lane()
{
    const int lane = __lane_id();
    return __builtin_amdgcn_readfirstlane(lane) == lane;
}

// Sum a per-lane counter over the wave and add it to a global total.
__device__ __forceinline__ void flush_work(const Work &w, uint64_t *work)
{
    uint32_t v[8] = {w.box, w.prism, w.edges, w.inserts, w.nodes, w.units, w.spills, w.leaves};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        uint64_t s = v[c];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
        if ((tid() & 63) == 0 && s) atomicAdd((unsigned long long *)&work[c], (unsigned long long)s);
    }
}

// One entry of a wave's traversal stack: a deferred node and the mask of
// the lanes that reached it.
struct alignas(16) StackEntry {
    int32_t node;
    uint32_t lo, hi, pad;
};

__device__ __forceinline__ uint64_t uniform64(uint32_t lo, uint32_t hi)
{
    const uint32_t l = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    const uint32_t h = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
    return ((uint64_t)h << 32) | l;
}

// Sum of v over all 64 lanes, returned to every lane; call with every lane
// of the wave active.  Quad permutes and row rotations (DPP, no LDS round
// trips) leave each 16-lane row's sum in all its lanes; the four row sums
// are read out and added.
template <int kCtrl>
__device__ __forceinline__ float add_dpp(float x)
{
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, false));
}

__device__ __forceinline__ float wave_sum(float v)
{
    v = add_dpp<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = add_dpp<0x4E>(v);   // quad_perm [2, 3, 0, 1]: quad sums
    v = add_dpp<0x124>(v);  // row_ror 4: two quads
    v = add_dpp<0x128>(v);  // row_ror 8: the row
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

// Is this lane's bit set in a wave-uniform mask?  (maps to the exec mask)
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Scalar helpers of the traversal loops.  Written as compare-and-selects
// on 64-bit lane masks: the compiler otherwise turns these conditions into
// lane-mask booleans and spends three or four extra scalar instructions
// per node on them.
// defer = h0 != 0 ? h1 : 0 (the second child, when both are wanted)
__device__ __forceinline__ uint64_t defer_mask(uint64_t h0, uint64_t h1)
{
    uint64_t d;
    asm("s_cmp_lg_u64 %[h0], 0\n"
        "s_cselect_b64 %[d], %[h1], 0"
        : [d] "=&s"(d)
        : [h0] "s"(h0), [h1] "s"(h1)
        : "scc");
    return d;
}
// (node, cur) = h0 != 0 ? (r0, h0) : (r1, h1) (the first child wanted)
__device__ __forceinline__ void descend(uint64_t h0, uint64_t h1, int r0, int r1, int &node, uint64_t &cur)
{
    asm("s_cmp_lg_u64 %[h0], 0\n"
        "s_cselect_b32 %[n], %[r0], %[r1]\n"
        "s_cselect_b64 %[c], %[h0], %[h1]"
        : [n] "=&s"(node), [c] "=&s"(cur)
        : [h0] "s"(h0), [h1] "s"(h1), [r0] "s"(r0), [r1] "s"(r1)
        : "scc");
}

// Packet traversal.  `bt(x0, y0, x1, y1, z1)` is the per-lane child-box
// test (a bool, or directly the lane mask of the lanes that pass);
// `leaf(prim, voff, m, want)` processes a leaf for the lanes in the mask
// `want` and returns the mask of lanes it retires.  `key(x0,y0,x1,y1,z1)`
// orders two wanted children (smaller first).  The walk starts with the
// lanes in `alive` and ends when none is left or the stack runs dry.  A
// lane only tests the children of nodes it reached itself: the walk
// carries the wave mask of the lanes that reached the current node, and
// every stack entry keeps the mask of the lanes that wanted it, so leaves
// no lane reached are skipped.  All the bookkeeping is on those
// wave-uniform masks (scalar registers; liveness too, so no per-lane flag
// is carried around the loop); the only per-lane work is the box tests.
// With kCount, `w` accumulates those box tests and the wave's node
// fetches.
template <bool kCount, class BoxTest, class LeafFn, class KeyFn>
__device__ __forceinline__ void packet_traverse(cNode *nodes, StackEntry *stack, uint64_t alive, BoxTest bt,
                                                LeafFn leaf, KeyFn key, Work &w)
{
    typedef __attribute__((address_space(4))) const char cchar;
    uint64_t cur = alive;
    int sp = 0, node = 0;
    while (cur) {
        // 64-byte nodes: a shifted index is the register offset of one
        // scalar load
        const Node nd = ld((cNode *)((cchar *)nodes + ((uint32_t)node << 6)));
        if constexpr (kCount) {
            w.box += lane_in(cur) ? 2u : 0u;
            w.nodes += first_active_lane() ? 1u : 0u;
        }
        uint64_t h0 = to_mask(bt(nd.lx0, nd.ly0, nd.lx1, nd.ly1, nd.lz1)) & cur;
        uint64_t h1 = to_mask(bt(nd.rx0, nd.ry0, nd.rx1, nd.ry1, nd.rz1)) & cur;
        int r0 = nd.left, r1 = nd.right;
        if ((r0 | r1) < 0) {
            // a leaf child, or the absent right child of a one-prism
            // hierarchy
            uint64_t out = 0;
            if (r0 < 0) {
                if (h0 && r0 != kNone) out |= leaf(~r0, nd.l_voff, nd.l_m, h0);
                h0 = 0;
            }
            if (r1 < 0) {
                if (h1 && r1 != kNone) out |= leaf(~r1, nd.r_voff, nd.r_m, h1);
                h1 = 0;
            }
            alive &= ~out;
            h0 &= alive;
            h1 &= alive;
        }
        if (h0 && h1) {
            // the visiting order must be one decision for the whole wave:
            // with per-lane keys (lanes on different segments) lanes could
            // disagree and the shared stack would lose a subtree
            const bool rfirst = uniform(key(nd.lx0, nd.ly0, nd.lx1, nd.ly1, nd.lz1) >
                                        key(nd.rx0, nd.ry0, nd.rx1, nd.ry1, nd.rz1)) != 0;
            if (rfirst) {
                const uint64_t th = h0;
                h0 = h1;
                h1 = th;
                const int tr = r0;
                r0 = r1;
                r1 = tr;
            }
        }
        const uint64_t defer = defer_mask(h0, h1);
        if (defer) {
            stack[sp] = StackEntry{r1, (uint32_t)defer, (uint32_t)(defer >> 32), 0u};
            ++sp;
        }
        descend(h0, h1, r0, r1, node, cur);
        if (!cur) {
            const uint64_t keep = alive;
            while (sp > 0) {
                --sp;
                const StackEntry e = stack[sp];
                node = uniform(e.node);
                cur = uniform64(e.lo, e.hi) & keep;
                if (cur) break;
            }
        }
    }
}

// Closed convex prism vs the ray p + s d (s > 0): clip the ray's footprint
// projection by every edge half-plane (Cyrus-Beck) in coordinates relative
// to p, then compare the height where it enters with the roof.
__device__ __forceinline__ bool ray_prism(cfloat4 *verts, int voff, int m, float H, float px, float py,
                                          float pz, float dx, float dy, float dz)
{
    float s_in = -INFINITY, s_out = INFINITY;
    for (int e = 0; e < m; ++e) {
        const float4 v = ld(verts + voff + e);
        const float wx = v.x - px, wy = v.y - py;
        const float num = fmaf(v.z, wx, v.w * wy);
        const float den = fmaf(v.z, dx, v.w * dy);   // the same for every lane
        const float s = num * __builtin_amdgcn_rcpf(den);
        // selects, not branches (see packet_traverse)
        s_out = den > 0.f ? fminf(s_out, s) : s_out;
        s_in = den < 0.f ? fmaxf(s_in, s) : s_in;
        s_out = ((den == 0.f) & (num < 0.f)) ? -INFINITY : s_out;
    }
    const float s0 = fmaxf(s_in, 0.f);
    return (s_out >= s0) & (fmaf(s0, dz, pz) <= H);
}

// Is (px, py) inside (or on) the convex CCW footprint?
__device__ __forceinline__ bool in_footprint(cfloat4 *verts, int voff, int m, float px, float py)
{
    bool in = true;
    for (int e = 0; e < m; ++e) {
        const float4 v = ld(verts + voff + e);
        // v.z, v.w = outward normal of the edge from this vertex
        in = in && fmaf(v.z, px - v.x, v.w * (py - v.y)) <= 0.f;
    }
    return in;
}

// ---- angles and directions of the segment geometry, written out so that
// the kernels make no library calls (a call imposes the calling convention
// on the whole kernel: registers saved and reloaded around every site) ----

// atan on [0, 1].  Above tan(pi/8) the reflection
// atan(t) = pi/4 + atan((t - 1) / (t + 1)) brings the argument to
// |u| <= tan(pi/8); there the Taylor series u - u^3/3 + ... - u^15/15 +
// u^17/17 is within |u|^19/19 < 3e-9 of atan(u).
__device__ __forceinline__ float atan01(float t)
{
    const bool refl = t > 0.41421356f;
    const float u = refl ? (t - 1.f) * __builtin_amdgcn_rcpf(t + 1.f) : t;
    const float s = u * u;
    float p = 1.f / 17.f;
    p = fmaf(p, s, -1.f / 15.f);
    p = fmaf(p, s, 1.f / 13.f);
    p = fmaf(p, s, -1.f / 11.f);
    p = fmaf(p, s, 1.f / 9.f);
    p = fmaf(p, s, -1.f / 7.f);
    p = fmaf(p, s, 1.f / 5.f);
    p = fmaf(p, s, -1.f / 3.f);
    p = fmaf(p, s, 1.f);
    const float r = u * p;
    return refl ? r + 0.785398163f : r;
}

// Polar angle of (x, y) in [-pi, pi] (atan2(y, x)), by the octant
// symmetries atan(y/x) = pi/2 - atan(x/y) and pi - angle for x < 0.
__device__ __forceinline__ float polar_angle(float x, float y)
{
    const float ax = fabsf(x), ay = fabsf(y);
    const float mx = fmaxf(ax, ay), mn = fminf(ax, ay);
    const float t = mx > 0.f ? fminf(mn * __builtin_amdgcn_rcpf(mx), 1.f) : 0.f;
    float r = atan01(t);
    r = ay > ax ? 1.57079633f - r : r;
    r = x < 0.f ? 3.14159265f - r : r;
    return y < 0.f ? -r : r;
}

// sin and cos of an angle in [0, 2 pi): w = k pi/2 + r with |r| <= pi/4
// (pi/2 split in two parts, Cody and Waite, so k pi/2 is subtracted
// without cancellation), Taylor series of sin to r^9 and cos to r^10
// (truncation below 2e-9), then the quadrant k.
__device__ __forceinline__ void sincos_small(float w, float &sn, float &cs)
{
    const float k = rintf(w * 0.636619772f);
    float r = fmaf(-k, 1.5703125f, w);
    r = fmaf(-k, 4.83826794897e-4f, r);
    const float z = r * r;
    float ps = -1.f / 362880.f;
    ps = fmaf(ps, z, 1.f / 5040.f);
    ps = fmaf(ps, z, -1.f / 120.f);
    ps = fmaf(ps, z, 1.f / 6.f);
    const float s = fmaf(-r * z, ps, r);
    float pc = -1.f / 3628800.f;
    pc = fmaf(pc, z, 1.f / 40320.f);
    pc = fmaf(pc, z, -1.f / 720.f);
    pc = fmaf(pc, z, 1.f / 24.f);
    pc = fmaf(pc, z, -0.5f);
    const float c = fmaf(pc, z, 1.f);
    const int q = (int)k & 3;
    sn = q == 0 ? s : (q == 1 ? c : (q == 2 ? -s : -c));
    cs = q == 0 ? c : (q == 1 ? -s : (q == 2 ? -c : s));
}

// ---- sorted disjoint interval set of at most 4 members, in registers ----
struct Union4 {
    float lo[4], hi[4];
    int n;
};

__device__ __forceinline__ void union_clear(Union4 &U)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) U.lo[i] = U.hi[i] = 0.f;
    U.n = 0;
}

// Insert the closed interval [a, b]; false if the result would need more
// than four disjoint members (the set is left unchanged).
__device__ __forceinline__ bool union_insert(Union4 &U, float a, float b)
{
    int nb = 0, na = 0;
    float mlo = a, mhi = b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool use = i < U.n;
        const bool before = use && U.hi[i] < a;
        const bool after = use && U.lo[i] > b;
        const bool ov = use && !before && !after;
        nb += before;
        na += after;
        mlo = ov ? fminf(mlo, U.lo[i]) : mlo;
        mhi = ov ? fmaxf(mhi, U.hi[i]) : mhi;
    }
    const int k = U.n - nb - na;
    const int nn = nb + 1 + na;
    if (nn > 4) return false;
    float nlo[4], nhi[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int src = j - 1 + k;
        float slo = U.lo[0], shi = U.hi[0];
#pragma unroll
        for (int s = 1; s < 4; ++s) {
            slo = src == s ? U.lo[s] : slo;
            shi = src == s ? U.hi[s] : shi;
        }
        nlo[j] = j < nb ? U.lo[j] : (j == nb ? mlo : slo);
        nhi[j] = j < nb ? U.hi[j] : (j == nb ? mhi : shi);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        U.lo[j] = nlo[j];
        U.hi[j] = nhi[j];
    }
    U.n = nn;
    return true;
}

// The same for sets known to be empty, and for sets of at most one member.
__device__ __forceinline__ void union_first(Union4 &U, float a, float b)
{
    U.lo[0] = a;
    U.hi[0] = b;
    U.n = 1;
}

__device__ __forceinline__ void union_second(Union4 &U, float a, float b)
{
    const bool one = U.n > 0;
    const bool before = one && U.hi[0] < a, after = one && U.lo[0] > b;
    const bool ov = one && !before && !after;
    U.lo[1] = before ? a : U.lo[0];
    U.hi[1] = before ? b : U.hi[0];
    U.lo[0] = before ? U.lo[0] : (ov ? fminf(a, U.lo[0]) : a);
    U.hi[0] = before ? U.hi[0] : (ov ? fmaxf(b, U.hi[0]) : b);
    U.n = (before || after) ? 2 : 1;
}

// Insert [a, b] for the lanes of the wave mask `in`; returns those whose set
// would need more than four members (left unchanged).  Most sets have no
// member or one when the next interval arrives, so the wave takes the
// shortest code that fits all of its lanes: a general insertion is about 100
// VALU instructions, the others 3 and 15.  With the shared polar_angle of
// prism_interval this took the block scene's accrual (4M points, three days)
// from 11.06 to 10.26 ms and 1-minute knots on 200k points, forward and
// adjoint, from 10.95 to 10.10 ms.
__device__ __forceinline__ uint64_t union_insert_mask(Union4 &U, float a, float b, uint64_t in)
{
    uint64_t over = 0;
    if (in & ballot(U.n > 1)) {
        bool o = false;
        if (lane_in(in)) o = !union_insert(U, a, b);
        over = ballot(o);
    } else if (in & ballot(U.n > 0)) {
        if (lane_in(in)) union_second(U, a, b);
    } else {
        if (lane_in(in)) union_first(U, a, b);
    }
    return over;
}

__device__ __forceinline__ float cross2(float au, float av, float bu, float bv)
{
    return fmaf(au, bv, -av * bu);
}

// Occluded angle interval of one prism over the window [w0, w1] of a
// segment, for a point at p.  In the segment's plane through p the prism
// is a convex polygon: the footprint lifted vertically into the plane and
// clipped to heights <= H.  The directions from p that meet it form one
// angular interval of span < pi (p is outside); its ends are found by
// cross products over the clipped polygon's vertices (the kept footprint
// vertices and the two clip crossings), and intersected with the window.
// `lanes`: the wave mask of the lanes asking; returns the mask of those with
// an overlap, whose [a, b] is written.  (Run by every lane of the traversal:
// all control is on masks, and candidates of other lanes are left out of it.)
//
// The lift of a horizontal offset w into the plane divides by the plane
// normal's vertical part nz, which vanishes for a plane through the
// zenith.  Only directions from p matter, so the segment's map M (and the
// heights it gives) carries the factor |nz|: vertices stay bounded for
// every plane, and the clip compares scaled heights with |nz| (H - pz).
// A clip crossing lies at height H - pz itself, so its in-plane point is
// formed directly from its world offset c as (e1 . (c, H - pz),
// e2 . (c, H - pz)), which has no cancellation when nz is small.
//
// With kGrad, da / db receive d(a)/dH and d(b)/dH: an end at a clip
// crossing moves with the roof along the lifted edge, dc/dH = (c1 - c0) /
// (z1 - z0) (the scale cancels), so d(angle)/dH = cross(c, c1 - c0) /
// (|c|^2 (z1 - z0)); ends at footprint vertices (vertical edges) or
// clamped to the window do not move.
template <bool kGrad>
__device__ __forceinline__ uint64_t prism_interval(cfloat4 *verts, int voff, int m, float H, uint64_t lanes, float px,
                                                   float py, float pz, const SegConst &g, float w0, float w1,
                                                   float W0u, float W0v, float W1u, float W1v, float &a, float &b,
                                                   float &da, float &db)
{
    const float h = H - pz;
    const float hs = h * fabsf(g.nz);  // the clip height in the scaled plane
    float lou = 0.f, lov = 0.f, hiu = 0.f, hiv = 0.f, dlo = 0.f, dhi = 0.f;
    // Lane masks (scalar registers) for the per-lane flags: which lanes have
    // a candidate yet, which see the footprint from inside every edge, which
    // vertices are below the roof line.  Only the selects are vector work.
    uint64_t have = 0, inside = ~0ull;
    if (kGrad || g.steep) {
        // extremes tracked in in-plane coordinates (derivatives, or a plane
        // too close to vertical for the world-offset shortcut below)
        auto cand = [&](float cu, float cv, float dc, uint64_t ok) {
            const uint64_t take_lo = ok & (~have | lt_mask(cross2(lou, lov, cu, cv), 0.f));
            const uint64_t take_hi = ok & (~have | gt_mask(cross2(hiu, hiv, cu, cv), 0.f));
            lou = lane_in(take_lo) ? cu : lou;
            lov = lane_in(take_lo) ? cv : lov;
            hiu = lane_in(take_hi) ? cu : hiu;
            hiv = lane_in(take_hi) ? cv : hiv;
            if constexpr (kGrad) {
                dlo = lane_in(take_lo) ? dc : dlo;
                dhi = lane_in(take_hi) ? dc : dhi;
            }
            have |= ok;
        };
        const float e1h = g.e1z * h, e2h = g.e2z * h;
        // footprint vertex k relative to p: world offset (wx, wy), scaled
        // in-plane (u, v) and scaled height z of the plane above p there
        auto vertex = [&](int k, float &wx, float &wy, float &u, float &v, float &z) {
            const float4 q = ld(verts + voff + k);
            wx = q.x - px;
            wy = q.y - py;
            u = fmaf(g.m00, wx, g.m01 * wy);
            v = fmaf(g.m10, wx, g.m11 * wy);
            z = fmaf(g.e1z, u, g.e2z * v);
        };
        // edge from vertex A to vertex B (world offsets, scaled in-plane
        // coordinates and heights, below-roof masks); returns the lanes for
        // which the edge faces away from p
        auto edge = [&](float awx, float awy, float au, float av, float az, uint64_t ain, float bwx, float bwy,
                        float bu, float bv, float bz, uint64_t bin) -> uint64_t {
            const uint64_t back = ge_mask(cross2(awx, awy, bwx, bwy), 0.f);
            inside &= back;
            const uint64_t crossing = (ain ^ bin) & lanes;
            if (crossing) {
                const float rdz = __builtin_amdgcn_rcpf(bz - az);
                const float t = (hs - az) * rdz;
                const float cx = fmaf(t, bwx - awx, awx), cy = fmaf(t, bwy - awy, awy);
                const float cu = fmaf(g.e1x, cx, fmaf(g.e1y, cy, e1h));
                const float cv = fmaf(g.e2x, cx, fmaf(g.e2y, cy, e2h));
                float dc = 0.f;
                if constexpr (kGrad)
                    dc = cross2(cu, cv, bu - au, bv - av) * rdz * __builtin_amdgcn_rcpf(fmaf(cu, cu, cv * cv));
                cand(cu, cv, dc, crossing);
            }
            return back;
        };
        // kept vertices: candidates only at the silhouette (see the
        // world-offset branch below)
        auto vcand = [&](float u, float v, uint64_t in, uint64_t b_in, uint64_t b_out) {
            const uint64_t ok = in & (b_in ^ b_out) & lanes;
            if (ok) cand(u, v, 0.f, ok);
        };
        // two vertices per trip, as in the world-offset branch below
        float awx, awy, au, av, az, bwx, bwy, bu, bv, bz;
        vertex(0, awx, awy, au, av, az);
        uint64_t ain = le_mask(az, hs);
        vertex(1, bwx, bwy, bu, bv, bz);
        uint64_t bin = le_mask(bz, hs);
        const uint64_t back0 = edge(awx, awy, au, av, az, ain, bwx, bwy, bu, bv, bz, bin);
        uint64_t bprev = back0;
        int e = 2;
        for (; e + 1 < m; e += 2) {
            vertex(e, awx, awy, au, av, az);
            ain = le_mask(az, hs);
            uint64_t back = edge(bwx, bwy, bu, bv, bz, bin, awx, awy, au, av, az, ain);
            vcand(bu, bv, bin, bprev, back);
            bprev = back;
            vertex(e + 1, bwx, bwy, bu, bv, bz);
            bin = le_mask(bz, hs);
            back = edge(awx, awy, au, av, az, ain, bwx, bwy, bu, bv, bz, bin);
            vcand(au, av, ain, bprev, back);
            bprev = back;
        }
        if (e < m) {  // one vertex left before the closing edge
            vertex(e, awx, awy, au, av, az);
            ain = le_mask(az, hs);
            const uint64_t back = edge(bwx, bwy, bu, bv, bz, bin, awx, awy, au, av, az, ain);
            vcand(bu, bv, bin, bprev, back);
            bprev = back;
            bwx = awx;
            bwy = awy;
            bu = au;
            bv = av;
            bz = az;
            bin = ain;
        }
        vertex(0, awx, awy, au, av, az);
        ain = le_mask(az, hs);
        const uint64_t bclose = edge(bwx, bwy, bu, bv, bz, bin, awx, awy, au, av, az, ain);
        vcand(bu, bv, bin, bprev, bclose);
        vcand(au, av, ain, bclose, back0);
    } else {
        // Without derivatives the extremes are found in world offsets from p:
        // the map M into the segment plane is linear, so it keeps the angular
        // order of directions (reverses it when det M < 0), and only the two
        // extremes are mapped at the end.  z, the plane's (scaled) height
        // above p at a footprint point, is linear in the offset too:
        // z = Z1 wx + Z2 wy.
        const float Z1 = fmaf(g.e1z, g.m00, g.e2z * g.m10), Z2 = fmaf(g.e1z, g.m01, g.e2z * g.m11);
        float lox = 0.f, loy = 0.f, hix = 0.f, hiy = 0.f;
        auto cand = [&](float cx, float cy, uint64_t ok) {
            const uint64_t take_lo = ok & (~have | lt_mask(cross2(lox, loy, cx, cy), 0.f));
            const uint64_t take_hi = ok & (~have | gt_mask(cross2(hix, hiy, cx, cy), 0.f));
            lox = lane_in(take_lo) ? cx : lox;
            loy = lane_in(take_lo) ? cy : loy;
            hix = lane_in(take_hi) ? cx : hix;
            hiy = lane_in(take_hi) ? cy : hiy;
            have |= ok;
        };
        auto vertex = [&](int k, float &wx, float &wy, float &z) {
            const float4 q = ld(verts + voff + k);
            wx = q.x - px;
            wy = q.y - py;
            z = fmaf(Z1, wx, Z2 * wy);
        };
        // Edge from vertex (ax, ay) (height az, below the roof line in the
        // lanes of ain) to vertex (bx, by, bz, bin); returns the lanes for
        // which the edge faces away from p (p on its inner side).
        auto edge = [&](float ax, float ay, float az, uint64_t ain, float bx, float by, float bz,
                        uint64_t bin) -> uint64_t {
            const uint64_t back = ge_mask(cross2(ax, ay, bx, by), 0.f);
            inside &= back;
            const uint64_t crossing = (ain ^ bin) & lanes;
            if (crossing) {
                const float t = (hs - az) * __builtin_amdgcn_rcpf(bz - az);
                cand(fmaf(t, bx - ax, ax), fmaf(t, by - ay, ay), crossing);
            }
            return back;
        };
        // Seen from p outside it, a convex polygon's extreme directions are
        // at its silhouette vertices, where the edge before and the edge
        // after face p differently.  The clipped polygon's edges at a kept
        // footprint vertex lie on the footprint's own edges, so a kept
        // vertex is a candidate only where the two footprint edges at it
        // disagree (the clip crossings are always candidates).  A vertex is
        // weighed once its outgoing edge is known; a vertex no lane needs
        // is skipped for the whole wave.
        auto vcand = [&](float x, float y, uint64_t in, uint64_t b_in, uint64_t b_out) {
            const uint64_t ok = in & (b_in ^ b_out) & lanes;
            if (ok) cand(x, y, ok);
        };
        // Two vertices per trip (A, then B, then A again), so the previous
        // vertex never has to be copied between registers; vertex 0 is read
        // again for the closing edge rather than kept in registers.
        float ax, ay, az, bx, by, bz;
        vertex(0, ax, ay, az);
        uint64_t ain = le_mask(az, hs);
        vertex(1, bx, by, bz);
        uint64_t bin = le_mask(bz, hs);
        const uint64_t back0 = edge(ax, ay, az, ain, bx, by, bz, bin);  // edge 0 -> 1
        uint64_t bprev = back0;
        int e = 2;
        for (; e + 1 < m; e += 2) {
            vertex(e, ax, ay, az);
            ain = le_mask(az, hs);
            uint64_t back = edge(bx, by, bz, bin, ax, ay, az, ain);
            vcand(bx, by, bin, bprev, back);
            bprev = back;
            vertex(e + 1, bx, by, bz);
            bin = le_mask(bz, hs);
            back = edge(ax, ay, az, ain, bx, by, bz, bin);
            vcand(ax, ay, ain, bprev, back);
            bprev = back;
        }
        if (e < m) {  // one vertex left before the closing edge
            vertex(e, ax, ay, az);
            ain = le_mask(az, hs);
            const uint64_t back = edge(bx, by, bz, bin, ax, ay, az, ain);
            vcand(bx, by, bin, bprev, back);
            bprev = back;
            bx = ax;
            by = ay;
            bz = az;
            bin = ain;
        }
        vertex(0, ax, ay, az);
        ain = le_mask(az, hs);
        const uint64_t bclose = edge(bx, by, bz, bin, ax, ay, az, ain);  // edge m-1 -> 0
        vcand(bx, by, bin, bprev, bclose);
        vcand(ax, ay, ain, bclose, back0);
        const bool flip = fmaf(g.m00, g.m11, -g.m01 * g.m10) < 0.f;
        const float fx = flip ? hix : lox, fy = flip ? hiy : loy;
        const float gx = flip ? lox : hix, gy = flip ? loy : hiy;
        lou = fmaf(g.m00, fx, g.m01 * fy);
        lov = fmaf(g.m10, fx, g.m11 * fy);
        hiu = fmaf(g.m00, gx, g.m01 * gy);
        hiv = fmaf(g.m10, gx, g.m11 * gy);
    }
    // Which ends lie inside the window: both directions of the window's ends
    // inside the interval need no angle; a lane asks for the angle of one end
    // in nearly every other case, so one polar_angle serves the lanes that
    // need the low end and those that need the high one.
    inside &= lanes;
    have &= ~inside;
    const uint64_t lo1 = ge_mask(cross2(lou, lov, W1u, W1v), 0.f);
    const uint64_t in0 = have & ge_mask(cross2(lou, lov, W0u, W0v), 0.f) & ge_mask(cross2(W0u, W0v, hiu, hiv), 0.f);
    const uint64_t in1 = have & lo1 & ge_mask(cross2(W1u, W1v, hiu, hiv), 0.f);
    const uint64_t within = have & ~(in0 | in1) & lo1 & ge_mask(cross2(W0u, W0v, lou, lov), 0.f);
    const uint64_t want_lo = (in1 & ~in0) | within, want_hi = (in0 & ~in1) | within;
    a = w0;
    b = w1;
    da = db = 0.f;
    if (want_lo | want_hi) {
        const bool hi = lane_in(want_hi);
        const float phi = polar_angle(hi ? hiu : lou, hi ? hiv : lov);
        const float c = fminf(fmaxf(phi, w0), w1);
        b = hi ? c : w1;
        a = lane_in(want_lo & ~want_hi) ? c : w0;
        if constexpr (kGrad) {
            db = (hi && c == phi) ? dhi : 0.f;
            da = (lane_in(want_lo & ~want_hi) && c == phi) ? dlo : 0.f;
        }
        if (within) {
            const float plo = polar_angle(lou, lov);
            const float d = fminf(fmaxf(plo, w0), w1);
            a = lane_in(within) ? d : a;
            if constexpr (kGrad) da = lane_in(within) ? (d == plo ? dlo : 0.f) : da;
        }
    }
    return (inside & ge_mask(h, 0.f)) | in0 | in1 | within;
}

// ---- interval set that also remembers, for every boundary, the prism
// whose interval end it is and that end's d(angle)/dH ----
struct UnionG {
    float lo[4], hi[4], dlo[4], dhi[4];
    int plo[4], phi[4];
    int n;
};

__device__ __forceinline__ void union_clear(UnionG &U)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        U.lo[i] = U.hi[i] = U.dlo[i] = U.dhi[i] = 0.f;
        U.plo[i] = U.phi[i] = -1;
    }
    U.n = 0;
}

// As union_insert; a merged boundary keeps the owner of the extreme end
// (equal ends: the lower prism index, -1 for the wall term first).
__device__ __forceinline__ bool union_insert(UnionG &U, float a, float b, int pa, int pb, float da, float db)
{
    int nb = 0, na = 0;
    float mlo = a, mhi = b, mdlo = da, mdhi = db;
    int mplo = pa, mphi = pb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool use = i < U.n;
        const bool before = use && U.hi[i] < a;
        const bool after = use && U.lo[i] > b;
        const bool ov = use && !before && !after;
        nb += before;
        na += after;
        const bool tlo = ov && (U.lo[i] < mlo || (U.lo[i] == mlo && U.plo[i] < mplo));
        const bool thi = ov && (U.hi[i] > mhi || (U.hi[i] == mhi && U.phi[i] < mphi));
        mlo = tlo ? U.lo[i] : mlo;
        mdlo = tlo ? U.dlo[i] : mdlo;
        mplo = tlo ? U.plo[i] : mplo;
        mhi = thi ? U.hi[i] : mhi;
        mdhi = thi ? U.dhi[i] : mdhi;
        mphi = thi ? U.phi[i] : mphi;
    }
    const int k = U.n - nb - na;
    const int nn = nb + 1 + na;
    if (nn > 4) return false;
    UnionG R;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int src = j - 1 + k;
        float slo = U.lo[0], shi = U.hi[0], sdlo = U.dlo[0], sdhi = U.dhi[0];
        int splo = U.plo[0], sphi = U.phi[0];
#pragma unroll
        for (int s = 1; s < 4; ++s) {
            const bool q = src == s;
            slo = q ? U.lo[s] : slo;
            shi = q ? U.hi[s] : shi;
            sdlo = q ? U.dlo[s] : sdlo;
            sdhi = q ? U.dhi[s] : sdhi;
            splo = q ? U.plo[s] : splo;
            sphi = q ? U.phi[s] : sphi;
        }
        const bool keep = j < nb, mid = j == nb;
        R.lo[j] = keep ? U.lo[j] : (mid ? mlo : slo);
        R.hi[j] = keep ? U.hi[j] : (mid ? mhi : shi);
        R.dlo[j] = keep ? U.dlo[j] : (mid ? mdlo : sdlo);
        R.dhi[j] = keep ? U.dhi[j] : (mid ? mdhi : sdhi);
        R.plo[j] = keep ? U.plo[j] : (mid ? mplo : splo);
        R.phi[j] = keep ? U.phi[j] : (mid ? mphi : sphi);
    }
    R.n = nn;
    U = R;
    return true;
}

__device__ __forceinline__ void union_first(UnionG &U, float a, float b, int pa, int pb, float da, float db)
{
    U.lo[0] = a;
    U.hi[0] = b;
    U.plo[0] = pa;
    U.phi[0] = pb;
    U.dlo[0] = da;
    U.dhi[0] = db;
    U.n = 1;
}

__device__ __forceinline__ void union_second(UnionG &U, float a, float b, int pa, int pb, float da, float db)
{
    const bool one = U.n > 0;
    const bool before = one && U.hi[0] < a, after = one && U.lo[0] > b;
    const bool ov = one && !before && !after;
    U.lo[1] = before ? a : U.lo[0];
    U.hi[1] = before ? b : U.hi[0];
    U.plo[1] = before ? pa : U.plo[0];
    U.phi[1] = before ? pb : U.phi[0];
    U.dlo[1] = before ? da : U.dlo[0];
    U.dhi[1] = before ? db : U.dhi[0];
    const bool klo = before || (ov && (U.lo[0] < a || (U.lo[0] == a && U.plo[0] < pa)));
    const bool khi = before || (ov && (U.hi[0] > b || (U.hi[0] == b && U.phi[0] < pb)));
    U.lo[0] = klo ? U.lo[0] : a;
    U.dlo[0] = klo ? U.dlo[0] : da;
    U.plo[0] = klo ? U.plo[0] : pa;
    U.hi[0] = khi ? U.hi[0] : b;
    U.dhi[0] = khi ? U.dhi[0] : db;
    U.phi[0] = khi ? U.phi[0] : pb;
    U.n = (before || after) ? 2 : 1;
}

// As union_insert_mask; the interval is prism p's.
__device__ __forceinline__ uint64_t union_insert_mask(UnionG &U, float a, float b, int p, float da, float db, uint64_t in)
{
    uint64_t over = 0;
    if (in & ballot(U.n > 1)) {
        bool o = false;
        if (lane_in(in)) o = !union_insert(U, a, b, p, p, da, db);
        over = ballot(o);
    } else if (in & ballot(U.n > 0)) {
        if (lane_in(in)) union_second(U, a, b, p, p, da, db);
    } else {
        if (lane_in(in)) union_first(U, a, b, p, p, da, db);
    }
    return over;
}

// Facade point whose wall faces away from the sun: n . d(phi) <= 0 with
// d(phi) = cos(phi) e1 + sin(phi) e2.  Over a window narrower than pi the
// set is one interval.  W0, W1: the window's end directions in (u, v).
// Returns 0 or 1 with [a, b].
__device__ __forceinline__ int backface_interval(float nx, float ny, const SegConst &g, float w0, float w1,
                                                 float W0u, float W0v, float W1u, float W1v, float &a, float &b)
{
    const float A = fmaf(nx, g.e1x, ny * g.e1y), B = fmaf(nx, g.e2x, ny * g.e2y);
    const float f0 = fmaf(A, W0u, B * W0v), f1 = fmaf(A, W1u, B * W1v);
    const bool s0 = f0 <= 0.f, s1 = f1 <= 0.f;
    if (s0 && s1) {
        a = w0;
        b = w1;
        return 1;
    }
    if (!s0 && !s1) return 0;
    // zero of A cos + B sin inside the window (|phi| < pi/2 there, B != 0):
    // atan(-A / B), taken as the polar angle of (|B|, -A sign B)
    const float z = fminf(fmaxf(polar_angle(fabsf(B), B > 0.f ? -A : A), w0), w1);
    if (s0) {
        a = w0;
        b = z;
    } else {
        a = z;
        b = w1;
    }
    return 1;
}

// End directions of the window [w0, w1] of segment g in (u, v): exact
// constants for the whole segment, sincos only for sub-windows.
__device__ __forceinline__ void window_dirs(const SegConst &g, float w0, float w1, float &W0u, float &W0v,
                                            float &W1u, float &W1v)
{
    if (w0 == 0.f) {
        W0u = 1.f;
        W0v = 0.f;
    } else {
        sincos_small(w0, W0v, W0u);
    }
    if (w1 == g.theta) {
        W1u = g.cth;
        W1v = g.sth;
    } else {
        sincos_small(w1, W1v, W1u);
    }
}

struct PointArgs {
    int64_t n;
    const float *x, *y, *z, *nx, *ny;
    const int32_t *owner;
    const int32_t *rank;  // original id -> hierarchy position
    int32_t n_b;
};

struct LanePoint {
    float px, py, pz, nx, ny;
    int own;  // hierarchy position of the owner, -1 for ground points
};

__device__ __forceinline__ LanePoint load_point(const PointArgs &P, int64_t i, bool valid)
{
    LanePoint q{0.f, 0.f, 0.f, 0.f, 0.f, -1};
    if (valid) {
        q.px = P.x[i];
        q.py = P.y[i];
        q.pz = P.z[i];
        if (P.nx) q.nx = P.nx[i];
        if (P.ny) q.ny = P.ny[i];
        if (P.owner) {
            const int o = P.owner[i];
            q.own = (o >= 0 && o < P.n_b) ? P.rank[o] : -1;
        }
    }
    return q;
}

// A kernel argument parked in LDS and read back, wave-uniform, where a
// persistent loop needs it: the register allocator then has no reason to
// hold it in scalar registers across the traversal (where it would spill
// them to vector lanes and restore them on every node visit).  The volatile
// read keeps the compiler from hoisting the reload out of the loop.
typedef __attribute__((address_space(3))) int lds_int;

template <class T>
__device__ __forceinline__ void lds_park(lds_int *w, const T &v)
{
    static_assert(sizeof(T) % 4 == 0, "word-sized objects");
    const int *s = (const int *)&v;
#pragma unroll
    for (unsigned k = 0; k < sizeof(T) / 4; ++k) w[k] = s[k];
}

template <class T>
__device__ __forceinline__ T lds_uniform(const lds_int *w)
{
    static_assert(sizeof(T) % 4 == 0, "word-sized objects");
    T r;
    int *d = (int *)&r;
    const volatile lds_int *p = w;
#pragma unroll
    for (unsigned k = 0; k < sizeof(T) / 4; ++k) d[k] = __builtin_amdgcn_readfirstlane(p[k]);
    return r;
}

struct SpillArgs {
    int4 *out;           // the queue: its one-lane entries, then the whole ones (kSpillSingles)
    uint32_t *counters;  // their numbers, the overflow flag
    int32_t cap;         // whole entries
};

// Queues the lanes of a wave (point i each, 64 of one tile) whose sets over
// segment j are left to the spill launch, in entries of a point each while there
// is room for them, else in one: so a launch of kSpillWork cannot fill the queue.
// (Entries of a point alone, 4M of them for 5e8 point-segments, refused a city
// of thin towers that left one window in 77.)
__device__ __forceinline__ void spill_push(const SpillArgs &S, uint64_t lanes, int i, int j)
{
    const uint32_t n = (uint32_t)__builtin_popcountll(lanes);
    uint32_t base = 0;
    if ((tid() & 63) == 0) base = atomicAdd(S.counters, n);
    base = (uint32_t)uniform((int)base);
    const bool fits = base <= kSpillSingles - n;
    const uint32_t at = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
    // where they don't fit: empty ones to the end
    if (lane_in(lanes) && at < kSpillSingles) S.out[at] = make_int4(i, j, fits ? 1 : 0, 0);
    if (fits || (tid() & 63) != 0) return;
    const uint32_t slot = atomicAdd(S.counters + 1, 1u);
    if (slot < (uint32_t)S.cap)
        S.out[kSpillSingles + slot] = make_int4(i, j, (int)(uint32_t)lanes, (int)(uint32_t)(lanes >> 32));
    else
        atomicOr(S.counters + 2, 1u);
}

// The items of a spill launch, a wave each: entries of a point (`singles` of
// them), then the 64 places of the others.
__device__ __forceinline__ int64_t spill_items(const uint32_t *counters, int32_t cap, uint32_t &singles)
{
    const uint2 n = *(const uint2 *)counters;  // (one round trip: all that a launch without entries does)
    singles = min(n.x, kSpillSingles);
    return (int64_t)singles + 64 * (int64_t)min(n.y, (uint32_t)cap);
}

// Item t's segment; returns its point, or less than 0 where the place is empty.
__device__ __forceinline__ int spill_item(const int4 *queue, uint32_t singles, int64_t t, int &j)
{
    const bool single = t < singles;
    const uint32_t u = (uint32_t)(t - singles);
    const int4 e = queue[single ? (uint32_t)t : kSpillSingles + (u >> 6)];
    j = uniform(e.y);
    const int first = uniform(e.x), at = single ? 0 : uniform((int)(u & 63u));
    return (uniform64((uint32_t)e.z, (uint32_t)e.w) >> at) & 1ull ? first + at : -1;
}

// What a launch's persistent waves start from: an empty spill queue and work
// counters at zero, cleared by the kernel before it (thread t < 256 of it).
__device__ __forceinline__ void clear_state(const LaunchState &L, int64_t t)
{
    if (L.queue_lengths && t < 2) L.queue_lengths[t] = 0u;
    if (t < L.n_counters) L.counters[t] = 0u;
}

// A spilled window (or one's sub-window) taken 64 ways by a wave.
struct SpillWindow {
    float w0, w1;
    int level;
};
constexpr int kSpillLevels = 3;
constexpr int kSpillWait = 64 * kSpillLevels;  // each level leaves at most 64, one of which the next takes

// Lane l takes [w0 + l d, w0 + (l + 1) d]: neighbours share the same rounded
// boundary, the last lane ends exactly at the window's end.
__device__ __forceinline__ void spill_share(const SpillWindow &win, int lane, float &w0, float &w1)
{
    const float d = (win.w1 - win.w0) * (1.f / 64.f);
    w0 = lane == 0 ? win.w0 : fmaf((float)lane, d, win.w0);
    w1 = lane == 63 ? win.w1 : fmaf((float)(lane + 1), d, win.w0);
}

// Lines up the sub-windows of the lanes with `ov` and takes the next one in
// line; false when none is left.
__device__ __forceinline__ bool spill_next(SpillWindow *wait, int &waiting, bool ov, float w0, float w1,
                                           uint32_t *overflow, SpillWindow &win)
{
    const uint64_t m = ballot(ov);
    if (m && win.level + 1 < kSpillLevels) {
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (ov) wait[waiting + rank] = SpillWindow{w0, w1, win.level + 1};
        waiting += __builtin_popcountll(m);
    } else if (m && first_active_lane()) {
        atomicOr(overflow, 2u);  // unfinished work
    }
    if (waiting == 0) return false;
    --waiting;
    const SpillWindow next = wait[waiting];
    win.w0 = __int_as_float(uniform(__float_as_int(next.w0)));
    win.w1 = __int_as_float(uniform(__float_as_int(next.w1)));
    win.level = uniform(next.level);
    return true;
}

// Per-lane fan/box test of one segment: the fan of directions from p below
// height z1 projects on the ground to the triangle p, p + (z1 - pz) ua,
// p + (z1 - pz) ub (central projection maps the great-circle arc to a
// segment), so the box test is a 2D separating-axis test against that
// triangle: its bounding box and the normals of its two edges through p.
// (The third edge, at the far end, is left out: the bounding box already
// bounds the far end, and measured over the block scene the edge removes
// under 1% of the box hits for 23% of the test's arithmetic.)  For an edge
// with normal n the box point farthest along n is the corner picked by
// the signs of n, so max n.x over the box is
//     x1 max(nx,0) + x0 min(nx,0) + y1 max(ny,0) + y0 min(ny,0),
// a wave-uniform value (the box is the wave's) compared with the lane's n.p.

// The fan of a segment seen from the xy plane: over the segment the rays
// from p sweep the wedge between the horizontal offsets ua (first knot) and
// ub (last knot), reaching (z - pz) * u at height z.  Returned: the
// per-metre reach box [umnx, umxx] x [umny, umxy] of the wedge and the two
// inward edge normals na (of p -> ua) and nb (of p -> ub).  Uniform per
// segment.
struct FanGeom {
    float umnx, umxx, umny, umxy;
    float nax, nay, nbx, nby;
};

__device__ __forceinline__ FanGeom fan_geom(const SegConst &g)
{
    FanGeom f;
    f.umnx = fminf(0.f, fminf(g.ua_x, g.ub_x));
    f.umxx = fmaxf(0.f, fmaxf(g.ua_x, g.ub_x));
    f.umny = fminf(0.f, fminf(g.ua_y, g.ub_y));
    f.umxy = fmaxf(0.f, fmaxf(g.ua_y, g.ub_y));
    f.nax = -g.ua_y;
    f.nay = g.ua_x;  // inward normal of p -> A (toward B)
    if (fmaf(f.nax, g.ub_x, f.nay * g.ub_y) < 0.f) {
        f.nax = -f.nax;
        f.nay = -f.nay;
    }
    f.nbx = -g.ub_y;
    f.nby = g.ub_x;  // inward normal of p -> B (toward A)
    if (fmaf(f.nbx, g.ua_x, f.nby * g.ua_y) < 0.f) {
        f.nbx = -f.nbx;
        f.nby = -f.nby;
    }
    return f;
}

// Largest value of n . x over the box [x0, x1] x [y0, y1] (the corner the
// normal points to), for a wedge edge normal n.
__device__ __forceinline__ float box_reach(float x0, float y0, float x1, float y1, float nx, float ny)
{
    return fmaf(y0, fminf(ny, 0.f), fmaf(y1, fmaxf(ny, 0.f), fmaf(x0, fminf(nx, 0.f), x1 * fmaxf(nx, 0.f))));
}

// Visit order of the prisms of a segment's view: nearer along the horizontal
// direction of the mid-segment sun first.  Half sums: finite, as (mdx, mdy) is
// and neither above one, for every finite box, so the key is never a NaN and
// each prism has a place of its own.
__device__ __forceinline__ float seg_key(float x0, float y0, float x1, float y1, float mdx, float mdy)
{
    return fmaf(fmaf(0.5f, x0, 0.5f * x1), mdx, fmaf(0.5f, y0, 0.5f * y1) * mdy);
}

// ---- the fan test on a segment's view of the scene ----
//
// A direct fan test of a box (the wedge edges' box_reach against
// each lane's n . p, and the box against the fan's bounding box, whose
// corners move with the box top by the per-metre reach) spends most of its
// arithmetic on values that are the same for every lane.  CDNA has no
// scalar floating point, so those values would cost full vector
// instructions at every visit.  Moving the lane's
// terms to the other side of each inequality,
//   x1 >= px + (z1 - pz) umnx   <=>   x1 - z1 umnx >= px - pz umnx,
// leaves one side that depends only on (segment, box), computed once per
// segment for the whole scene (ViewEntry), and one that depends only on
// (segment, point), computed once per lane and segment (SegFan): a
// test becomes six compares.  (A box whose top is below pz has no compare of
// its own: the bounds shifted by its negative rise nearly always exclude it.
// On the block scene, half its points on facades, 1 in 8,500 more box tests
// pass.)  Both sides are rounded outward, so the
// test passes every box that meets the fan exactly (boxes only decide
// what is tested, never a result).

typedef __attribute__((address_space(4))) const ViewEntry cView;

__device__ __forceinline__ float round_up_rel(float v) { return v + fabsf(v) * 0x1p-22f; }
__device__ __forceinline__ float round_dn_rel(float v) { return v - fabsf(v) * 0x1p-22f; }

struct SegFan {
    float cxl, cxh, cyl, cyh, naP, nbP;

    __device__ __forceinline__ SegFan(const SegConst &g, float px, float py, float pz)
        : SegFan(fan_geom(g), px, py, pz)
    {
    }

    __device__ __forceinline__ SegFan(const FanGeom &f, float px, float py, float pz)
    {
        cxl = round_dn_rel(fmaf(-pz, f.umnx, px));
        cxh = round_up_rel(fmaf(-pz, f.umxx, px));
        cyl = round_dn_rel(fmaf(-pz, f.umny, py));
        cyh = round_up_rel(fmaf(-pz, f.umxy, py));
        naP = fmaf(f.nax, px, f.nay * py);
        nbP = fmaf(f.nbx, px, f.nby * py);
    }

    // The lanes of cur whose fan meets the entry's box.
    __device__ __forceinline__ uint64_t one(const ViewEntry &v, uint64_t cur) const
    {
        uint64_t sv, h;
        asm volatile(
            "s_mov_b64 %[sv], exec\n"
            "s_mov_b64 exec, %[cur]\n"
            "v_cmpx_ge_f32 vcc, %[a0], %[cxl]\n"
            "v_cmpx_le_f32 vcc, %[a1], %[cxh]\n"
            "v_cmpx_ge_f32 vcc, %[a2], %[cyl]\n"
            "v_cmpx_le_f32 vcc, %[a3], %[cyh]\n"
            "v_cmpx_ge_f32 vcc, %[a4], %[naP]\n"
            "v_cmpx_ge_f32 vcc, %[a5], %[nbP]\n"
            "s_mov_b64 %[h], exec\n"
            "s_mov_b64 exec, %[sv]\n"
            "s_nop 1\n"  // a lane read waits four states for compares into exec
            : [h] "=&s"(h), [sv] "=&s"(sv)
            : [cur] "s"(cur), [cxl] "v"(cxl), [cxh] "v"(cxh), [cyl] "v"(cyl), [cyh] "v"(cyh), [naP] "v"(naP),
              [nbP] "v"(nbP), [a0] "s"(v.c[0]), [a1] "s"(v.c[1]), [a2] "s"(v.c[2]), [a3] "s"(v.c[3]), [a4] "s"(v.c[4]),
              [a5] "s"(v.c[5])
            : "vcc");
        return h;
    }
};

// The extremes of SegFan's terms over the lanes of a mask: the weakest a box
// must meet to be met by any of their fans.  They lie in LDS, a slot per wave:
// scalar registers are what a walk has least of (as six of them they were
// spilled to lanes and read back for every test).
struct alignas(16) TileFan {
    float cxl, cxh, cyl, cyh, naP, nbP;
};

__device__ __forceinline__ void tile_fan(TileFan *out, const SegFan &f, uint64_t lanes)
{
    float a = f.cxl, b = f.cxh, c = f.cyl, d = f.cyh, e = f.naP, g = f.nbP;
    if (lanes != ~0ull) {
        const bool in = lane_in(lanes);
        a = in ? a : INFINITY;
        b = in ? b : -INFINITY;
        c = in ? c : INFINITY;
        d = in ? d : -INFINITY;
        e = in ? e : INFINITY;
        g = in ? g : INFINITY;
    }
    // six reductions side by side: each step reads what was written five
    // instructions before
#define SA_STEP(ctrl)                       \
    "v_min_f32_dpp %[a], %[a], %[a] " ctrl  \
    "v_max_f32_dpp %[b], %[b], %[b] " ctrl  \
    "v_min_f32_dpp %[c], %[c], %[c] " ctrl  \
    "v_max_f32_dpp %[d], %[d], %[d] " ctrl  \
    "v_min_f32_dpp %[e], %[e], %[e] " ctrl  \
    "v_min_f32_dpp %[g], %[g], %[g] " ctrl
    asm volatile("s_nop 4\n" SA_STEP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n")
                     SA_STEP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n")
                         SA_STEP("row_ror:4 row_mask:0xf bank_mask:0xf\n")
                             SA_STEP("row_ror:8 row_mask:0xf bank_mask:0xf\n")
                                 SA_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf\n")
                                     SA_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf\n") "s_nop 0"
                 : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [e] "+v"(e), [g] "+v"(g));
#undef SA_STEP
    if ((tid() & 63) == 63) *out = TileFan{a, b, c, d, e, g};
    // (the wave's other lanes read it: LDS keeps a wave's order, and so must
    // the compiler)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// An entry per lane: the lanes whose box is met.
__device__ __forceinline__ uint64_t tile_meets(const TileFan *tile, const float4 &u, const float4 &v)
{
    const TileFan f = *tile;
    uint64_t sv, h;
    asm volatile(
        "s_mov_b64 %[sv], exec\n"
        "v_cmpx_le_f32 vcc, %[cxl], %[a0]\n"
        "v_cmpx_ge_f32 vcc, %[cxh], %[a1]\n"
        "v_cmpx_le_f32 vcc, %[cyl], %[a2]\n"
        "v_cmpx_ge_f32 vcc, %[cyh], %[a3]\n"
        "v_cmpx_le_f32 vcc, %[naP], %[a4]\n"
        "v_cmpx_le_f32 vcc, %[nbP], %[a5]\n"
        "s_mov_b64 %[h], exec\n"
        "s_mov_b64 exec, %[sv]\n"
        "s_nop 1\n"  // a lane read waits four states for compares into exec
        : [h] "=&s"(h), [sv] "=&s"(sv)
        : [cxl] "v"(f.cxl), [cxh] "v"(f.cxh), [cyl] "v"(f.cyl), [cyh] "v"(f.cyh), [naP] "v"(f.naP), [nbP] "v"(f.nbP),
          [a0] "v"(u.x), [a1] "v"(u.y), [a2] "v"(u.z), [a3] "v"(u.w), [a4] "v"(v.x), [a5] "v"(v.y)
        : "vcc");
    return h;
}

// The box-only side of SegFan's inequalities for one child box.  The
// shifted edges are formed in double and rounded outward; the wedge
// projections are box_reach.  An absent child gets a box no
// lane passes.
__device__ __forceinline__ void seg_child(const FanGeom &f, float x0, float y0, float x1, float y1, float z1,
                                          bool present, float *c)
{
    if (!present) {
        c[0] = c[2] = c[4] = c[5] = -INFINITY;
        c[1] = c[3] = INFINITY;
        return;
    }
    c[0] = round_up_rel((float)((double)x1 - (double)z1 * f.umnx));
    c[1] = round_dn_rel((float)((double)x0 - (double)z1 * f.umxx));
    c[2] = round_up_rel((float)((double)y1 - (double)z1 * f.umny));
    c[3] = round_dn_rel((float)((double)y0 - (double)z1 * f.umxy));
    c[4] = box_reach(x0, y0, x1, y1, f.nax, f.nay);
    c[5] = box_reach(x0, y0, x1, y1, f.nbx, f.nby);
}

// A prism's vertex range in one word of its entry; 0 above kLeafVertBits where
// it does not fit.
__device__ __forceinline__ uint32_t leaf_word(int voff, int m)
{
    const bool fits = voff < (1 << kLeafVertBits) && m < (1 << (32 - kLeafVertBits));
    return fits ? (uint32_t)voff | (uint32_t)m << kLeafVertBits : 0u;
}

__device__ __forceinline__ void leaf_range(uint32_t word, cint *voff, int prim, int &v0, int &m)
{
    v0 = (int)(word & ((1u << kLeafVertBits) - 1u));
    m = (int)(word >> kLeafVertBits);
    if (m == 0) {
        v0 = ld(voff + prim);
        m = ld(voff + prim + 1) - v0;
    }
}

// A fan's walk over its view of the scene, for the lanes in `alive`: a lane
// takes an entry of a group at a time and tests its box against the tile's
// extremes, so 64 boxes cost six vector compares; only a prism that passes is
// tested by every lane for itself.  Groups lie in the view nearest along the
// fan's middle direction first (within 64), so shadowed lanes retire early.
// `leaf(prim, voff, m, want)` returns the mask of lanes it retires.  All 64
// lanes of the wave must be here: each stands for a box.
// Bound by VALU issue.  A binary tree with both children's boxes tested by
// every lane visited 26 nodes a wave and segment of the block scene (4M
// points, 20,000 prisms, three days); this makes 3 tests of groups, 1 or 2 of
// prisms and 3 of a single one: 10.07 -> 7.20 ms, VALU instructions 5.2e9 ->
// 4.1e9.  Also there: longest runs 1.77 -> 1.33 ms, the sampled form 4.96 ->
// 4.06; contributions 1.08 -> 0.88, forward and adjoint at 1-minute knots
// 10.1 -> 7.5, a year on 45,000 prisms 207 -> 143, small calls 0 to 20 % less.
// Groups in Morton order instead (whose runs jump, so far groups come before
// near ones): 10.0 ms, eight times the spilled sets.  The extremes in scalar
// registers and the shape held across the walk: 0.1 ms more.
// kBlocks: the scene has more than one block of groups of groups.  (Kernels are
// built for either: the blocks' part costs the others' registers, 2 to 5 % of
// every call on 5,000 and 20,000 prisms.)
template <bool kCount, bool kBlocks, class LeafFn>
__device__ __forceinline__ void walk_view(const ViewEntry *view, int n_b, cint *voff, TileFan *tile, uint64_t alive,
                                          const SegFan &ft, LeafFn leaf, Work &w)
{
    if (!alive) return;
    tile_fan(tile, ft, alive);
    const int lane = (int)(tid() & 63);
    // the shape is worked out where it is used, on the scalar unit, not held
    auto shape = [&]() {
        int n = n_b;
        asm volatile("" : "+s"(n));
        return view_shape<kBlocks>(n);
    };
    cView *cv = (cView *)view;
    auto test = [&](uint32_t at, int &ref) -> uint64_t {
        const char *e = (const char *)view + at * (uint32_t)sizeof(ViewEntry);
        if constexpr (kCount) {
            w.box += 1u;
            w.nodes += first_active_lane() ? 1u : 0u;
        }
        const float4 v = *(const float4 *)(e + 16);
        ref = __float_as_int(v.z);
        return tile_meets(tile, *(const float4 *)e, v);
    };
    auto first_of = [](int n) -> uint64_t { return n >= 64 ? ~0ull : (1ull << n) - 1ull; };
    int ref, none;
    // the k3-th block, nearest first; its number is read where it is used, and
    // what is left of its siblings found again after it, for registers' sake
    auto first_super = [&](const ViewShape &sh, int k3) { return sh.n3 > 1 ? ld(cv + k3).ref << kBlockBits : 0; };
    for (int k3 = 0;;) {
        ViewShape sh = shape();
        if (sh.n3 > 1) {
            const int c3 = k3 & ~63;
            const uint64_t m3 = test((uint32_t)min(c3 + lane, sh.n3 - 1), none) & first_of(sh.n3 - c3) & (~0ull << (k3 & 63));
            k3 = c3 + (m3 ? (int)__builtin_ctzll(m3) : 64);
            if (k3 >= sh.n3) break;
            if (!m3) continue;
        }
        uint64_t m2 = 1ull;
        if (sh.n2 > 1) {
            const int c2 = first_super(sh, k3);
            m2 = test(sh.at2 + (uint32_t)min(c2 + lane, sh.n2 - 1), none) & first_of(sh.n2 - c2);
        }
        while (m2) {
            sh = shape();
            const int b1 = sh.n2 > 1 ? ld(cv + sh.at2 + first_super(sh, k3) + (int)__builtin_ctzll(m2)).ref << kSuperBits : 0;
            m2 &= m2 - 1ull;
            uint64_t m1 = 1ull;
            if (sh.n1 > 1) m1 = test(sh.at1 + (uint32_t)min(b1 + lane, sh.n1 - 1), ref) & first_of(sh.n1 - b1);
            while (m1) {
                // two groups at a time, half a wave each
                sh = shape();
                const int ka = (int)__builtin_ctzll(m1);
                m1 &= m1 - 1ull;
                const int kb = m1 ? (int)__builtin_ctzll(m1) : ka;
                const uint64_t both = m1 ? ~0ull : 0xffffffffull;
                m1 &= m1 - 1ull;
                int fa = 0, fb = 0;  // their first prisms
                if (sh.n1 > 1) {
                    fa = __builtin_amdgcn_readlane(ref, ka) << kGroupBits;
                    fb = __builtin_amdgcn_readlane(ref, kb) << kGroupBits;
                }
                const int mine = (lane & 31) + (lane < 32 ? fa : fb);
                uint64_t m0 = test(sh.at0 + (uint32_t)min(mine, sh.n_b - 1), none) & both & ballot(mine < sh.n_b);
                cView *prisms = cv + sh.at0;
                while (m0) {
                    const int k = (int)__builtin_ctzll(m0);
                    m0 &= m0 - 1ull;
                    const ViewEntry v = ld(prisms + (k < 32 ? fa : fb) + (k & 31));
                    const uint64_t h = ft.one(v, alive);
                    if constexpr (kCount) {
                        w.box += lane_in(alive) ? 1u : 0u;
                        w.nodes += first_active_lane() ? 1u : 0u;
                    }
                    if (h) {
                        int v0, m;
                        leaf_range(v.vert, voff, v.ref, v0, m);
                        alive &= ~leaf(v.ref, v0, m, h);
                        m0 = alive ? m0 : 0ull;
                    }
                }
                m1 = alive ? m1 : 0ull;
            }
            m2 = alive ? m2 : 0ull;
        }
        // (a loop for one block too, to the compiler: without it the adjoint's
        // kernel keeps 41 registers in memory instead of 17, 6.36 -> 6.50 ms)
        int blocks = shape().n3;
        if constexpr (!kBlocks) asm volatile("" : "+s"(blocks));
        if (!alive || ++k3 >= blocks) break;
    }
}

// Footprint boxes of the prisms and of the views' groups (DeviceScene), for
// the roof test; n_b = 0: an empty scene.
struct RoofBoxes {
    const float4 *pbox, *gbox;
    const int32_t *vorder;
    int32_t n_b, pad;
};

// Roof-covered: inside a footprint (other than the point's own building)
// and not above that roof -- shadowed from every direction.  As walk_view, a
// lane takes a box: against the box of the wave's points, all 64 lanes here.
// Bound by its memory round trips, four where the binary hierarchy took one a
// level, once a unit: 16,384 points on 64 prisms 40.9 -> 38.4 us, 20,000 on 300
// 43.5 -> 39.1, 4M on 20,000 7.20 -> 7.00 ms, forward and adjoint at 1-minute
// knots 6.83 -> 6.67 ms.
template <bool kBlocks>
__device__ __forceinline__ bool roof_covered(const RoofBoxes &B, cint *voff, cfloat4 *verts, cfloat *height,
                                             const LanePoint &q, bool valid)
{
    const uint64_t asked = ballot(valid);
    if (B.n_b == 0 || !asked) return false;
    float x0 = valid ? q.px : INFINITY, x1 = valid ? q.px : -INFINITY;
    float y0 = valid ? q.py : INFINITY, y1 = valid ? q.py : -INFINITY;
    // (each step reads what was written three instructions before)
#define SA_STEP(ctrl)                          \
    "v_min_f32_dpp %[x0], %[x0], %[x0] " ctrl  \
    "v_max_f32_dpp %[x1], %[x1], %[x1] " ctrl  \
    "v_min_f32_dpp %[y0], %[y0], %[y0] " ctrl  \
    "v_max_f32_dpp %[y1], %[y1], %[y1] " ctrl
    asm volatile("s_nop 4\n" SA_STEP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n")
                     SA_STEP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n")
                         SA_STEP("row_ror:4 row_mask:0xf bank_mask:0xf\n")
                             SA_STEP("row_ror:8 row_mask:0xf bank_mask:0xf\n")
                                 SA_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf\n")
                                     SA_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf\n") "s_nop 0"
                 : [x0] "+v"(x0), [x1] "+v"(x1), [y0] "+v"(y0), [y1] "+v"(y1));
#undef SA_STEP
    auto last = [](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)); };
    const float X0 = last(x0), X1 = last(x1), Y0 = last(y0), Y1 = last(y1);
    auto meets = [&](const float4 &b) {
        return ballot(pad_lo(b.x) <= X1 && pad_hi(b.z) >= X0 && pad_lo(b.y) <= Y1 && pad_hi(b.w) >= Y0);
    };
    auto first_of = [](int n) -> uint64_t { return n >= 64 ? ~0ull : (1ull << n) - 1ull; };
    const ViewShape sh = view_shape<kBlocks>(B.n_b);
    const int lane = (int)(tid() & 63);
    uint64_t cov = 0;
    for (int c2 = 0; c2 < sh.n2; c2 += 64) {
        if (sh.n3 > 1) {
            // the next block that is met
            const int k3 = c2 >> kBlockBits, c3 = k3 & ~63;
            const uint64_t m3 = meets(B.gbox[sh.n1 + sh.n2 + min(c3 + lane, sh.n3 - 1)]) & first_of(sh.n3 - c3) & (~0ull << (k3 & 63));
            c2 = (c3 + (m3 ? (int)__builtin_ctzll(m3) : 63)) << kBlockBits;
            if (!m3) continue;
        }
        uint64_t m2 = 1ull;
        if (sh.n2 > 1) m2 = meets(B.gbox[sh.n1 + min(c2 + lane, sh.n2 - 1)]) & first_of(sh.n2 - c2);
        for (; m2; m2 &= m2 - 1ull) {
            const int b1 = (c2 + (int)__builtin_ctzll(m2)) << kSuperBits;
            uint64_t m1 = 1ull;
            if (sh.n1 > 1) m1 = meets(B.gbox[min(b1 + lane, sh.n1 - 1)]) & first_of(sh.n1 - b1);
            while (m1) {
                // two groups at a time, half a wave each
                const int ka = (int)__builtin_ctzll(m1);
                m1 &= m1 - 1ull;
                const int kb = m1 ? (int)__builtin_ctzll(m1) : ka;
                const uint64_t both = m1 ? ~0ull : 0xffffffffull;
                m1 &= m1 - 1ull;
                const int mine = ((b1 + (lane < 32 ? ka : kb)) << kGroupBits) + (lane & 31);
                const int prim = B.vorder[min(mine, B.n_b - 1)];
                const float4 box = B.pbox[prim];
                uint64_t m0 = meets(box) & both & ballot(mine < B.n_b);
                for (; m0; m0 &= m0 - 1ull) {
                    // few points lie in a box that their tile's meets
                    const int k = (int)__builtin_ctzll(m0);
                    const int b = __builtin_amdgcn_readlane(prim, k);
                    auto at = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k)); };
                    uint64_t want = asked & ~cov & ballot(b != q.own && q.px >= pad_lo(at(box.x)) && q.px <= pad_hi(at(box.z)) &&
                                                         q.py >= pad_lo(at(box.y)) && q.py <= pad_hi(at(box.w)));
                    if (!want) continue;
                    want &= ballot(q.pz <= ld(height + b));
                    const int v0 = ld(voff + b);
                    cov |= want & ballot(in_footprint(verts, v0, ld(voff + b + 1) - v0, q.px, q.py));
                }
            }
        }
    }
    return lane_in(cov);
}

}  // namespace dev
}  // namespace sa
