// Building the fans' views of a scene (ViewEntry).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>

#include "sa_internal.h"
#include "traverse.h"

namespace sa {
namespace dev {

__device__ __forceinline__ FanGeom fan_geom(const FanChunk &c)
{
    return FanGeom{c.f[0], c.f[1], c.f[2], c.f[3], c.f[4], c.f[5], c.f[6], c.f[7]};
}

constexpr int kViewThreads = 1024;
constexpr int kSuperPrisms = 1 << (kGroupBits + kSuperBits);

// Position of sibling k among its group's siblings (a key per lane, those of
// `in`), nearest first.
__device__ __forceinline__ int near_rank(float key, uint64_t in, int k)
{
    const float mine = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(key), k));
    const uint64_t before = ballot(key < mine) | (ballot(key == mine) & ((1ull << k) - 1ull));
    return __builtin_popcountll(before & in);
}

// Where a box begins along a direction.  A group comes where its near edge
// does: one that holds the points comes before those beyond, wherever its middle
// lies (by the middle 4,000 points among 15,000 prisms take 188 us, so 166; 4M
// among 20,000 in a strip 6.79 and 6.65 ms; a year of 16M points all over a city
// of 45,000 the other way, 5.0 and 5.9 s: there more sets spill, and keys in
// between lie in between).
__device__ __forceinline__ float near_edge(const float4 &q, float dx, float dy)
{
    return (dx > 0.f ? q.x : q.z) * dx + (dy > 0.f ? q.y : q.w) * dy;
}

// The first n lanes.
__device__ __forceinline__ uint64_t first_lanes(int n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; }

// Views of the scene for the fans [j0, ...) of a launch: one block per fan
// and group of groups, a thread per prism.  A wave's halves hold a group each,
// whose terms are reduced across them; the group's entry goes to its place by
// distance along the fan's middle direction, which every wave finds from the
// footprint boxes of the group's siblings (gbox).
// Bound by its writes: 32 bytes a prism and fan (64 a node before).
template <class Fan>
__global__ __launch_bounds__(kViewThreads) void k_views(const int32_t *__restrict__ vorder,
                                                        const float4 *__restrict__ pbox, const float *__restrict__ tops,
                                                        const float4 *__restrict__ gbox, const int32_t *__restrict__ voff,
                                                        int n_b, const Fan *__restrict__ fans, int j0,
                                                        ViewEntry *__restrict__ out, LaunchState L)
{
    __shared__ float s_max[kViewThreads / 64][6];
    clear_state(L, (int64_t)wg_id() * wg_size() + tid());
    const ViewShape sh = view_shape(n_b);
    const int jj = wg_id() / sh.n2, g2 = wg_id() - jj * sh.n2;
    const Fan &fan = fans[j0 + jj];
    const FanGeom f = fan_geom(fan);
    const float mdx = fan.mdx, mdy = fan.mdy;
    out += (int64_t)jj * sh.all;
    const int lane = (int)(tid() & 63);
    const int b1 = g2 << kSuperBits, b0 = g2 * kSuperPrisms;
    auto key_of = [&](const float4 &q) { return seg_key(q.x, q.y, q.z, q.w, mdx, mdy); };
    const float key1 = near_edge(gbox[min(b1 + lane, sh.n1 - 1)], mdx, mdy);
    const uint64_t in1 = first_lanes(sh.n1 - b1);
    // terms as maxima: the second and fourth negated
    float most[6] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY};
    const int end = min(n_b, b0 + kSuperPrisms);
    for (int at = b0 + (int)(tid() & ~63u); at < end; at += (int)wg_size()) {
        const int j = at + lane;
        const bool in = j < n_b;
        const int prim = vorder[min(j, n_b - 1)];
        const float4 q = pbox[prim];
        ViewEntry v;
        // (one variant's infinite height, or a padding past the largest float, must
        // not lose the prism to all of them: infinity times a reach of zero)
        const float top = fminf(pad_hi(tops[prim]), FLT_MAX);
        seg_child(f, pad_lo(q.x), pad_lo(q.y), pad_hi(q.z), pad_hi(q.w), top, in, v.c);
        // its place among its group's: how many are nearer
        const float key = key_of(q);
        const int left = n_b - at;  // of the wave's
        int nearer = 0;
#pragma unroll 8
        for (int o = 0; o < 32; ++o) {
            const float ka = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(key), o));
            const float kb = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(key), o + 32));
            const float k = lane < 32 ? ka : kb;
            const bool before = k < key || (k == key && o < (lane & 31));
            nearer += before && (lane & 32) + o < left ? 1 : 0;
        }
        if (in) {
            v.ref = prim;
            v.vert = leaf_word(voff[prim], voff[prim + 1] - voff[prim]);
            out[sh.at0 + (j & ~31) + nearer] = v;
        }
        if (sh.n1 == 1) continue;
        float m[6] = {v.c[0], -v.c[1], v.c[2], -v.c[3], v.c[4], v.c[5]};
#pragma unroll
        for (int k = 0; k < 6; ++k)
            for (int o = 1; o < 32; o <<= 1) m[k] = fmaxf(m[k], __shfl_xor(m[k], o, 64));
        const int ga = at >> kGroupBits;  // the first half's group
        const int ra = near_rank(key1, in1, ga - b1), rb = near_rank(key1, in1, min(ga + 1 - b1, 63));
        const int g = ga + (lane >> 5);
        if ((lane & 31) == 0 && g < sh.n1)
            out[sh.at1 + b1 + (lane ? rb : ra)] = ViewEntry{{m[0], -m[1], m[2], -m[3], m[4], m[5]}, g, 0u};
#pragma unroll
        for (int k = 0; k < 6; ++k) most[k] = fmaxf(most[k], m[k]);
    }
    if (sh.n2 == 1) return;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        most[k] = fmaxf(most[k], __shfl_xor(most[k], 32, 64));
        if (lane == 0) s_max[tid() >> 6][k] = most[k];
    }
    __syncthreads();
    if (tid() >= 64) return;
    // the first wave: this group of groups' entry among its block's
    const int c2 = g2 & ~63;
    const float key2 = near_edge(gbox[sh.n1 + min(c2 + lane, sh.n2 - 1)], mdx, mdy);
    const int r2 = near_rank(key2, first_lanes(sh.n2 - c2), g2 - c2);
    for (unsigned k = 0; k < 6; ++k) {
        float m = -INFINITY;
        for (unsigned w = 0; w < wg_size() / 64; ++w) m = fmaxf(m, s_max[w][k]);
        most[k] = m;
    }
    if (lane == 0)
        out[sh.at2 + c2 + r2] = ViewEntry{{most[0], -most[1], most[2], -most[3], most[4], most[5]}, g2, 0u};
}

// The entries of the blocks, from those of their groups of groups: a wave per
// fan and block.  Without them (groups of groups in the order of the curve, 64
// at a time) the points among a million prisms met far ones first: 1M points
// and 1M prisms 45 ms, 4M prisms 115.
template <class Fan>
__global__ __launch_bounds__(64) void k_view_blocks(const float4 *__restrict__ gbox, int n_b,
                                                    const Fan *__restrict__ fans, int j0, ViewEntry *__restrict__ out)
{
    const ViewShape sh = view_shape(n_b);
    const int jj = wg_id() / sh.n3, g = wg_id() - jj * sh.n3, lane = (int)tid();
    out += (int64_t)jj * sh.all;
    const ViewEntry e = out[sh.at2 + min((g << kBlockBits) + lane, sh.n2 - 1)];
    float most[6] = {e.c[0], -e.c[1], e.c[2], -e.c[3], e.c[4], e.c[5]};
#pragma unroll
    for (int k = 0; k < 6; ++k)
        for (int o = 1; o < 64; o <<= 1) most[k] = fmaxf(most[k], __shfl_xor(most[k], o, 64));
    const int c = g & ~63;
    const float key = near_edge(gbox[sh.n1 + sh.n2 + min(c + lane, sh.n3 - 1)], fans[j0 + jj].mdx, fans[j0 + jj].mdy);
    const int r = near_rank(key, first_lanes(sh.n3 - c), g - c);
    if (lane == 0) out[c + r] = ViewEntry{{most[0], -most[1], most[2], -most[3], most[4], most[5]}, g, 0u};
}

}  // namespace dev

// Launches k_views for the fans [j0, j1), and k_view_blocks.
template <class Fan>
static void launch_views(const DeviceScene &s, const float *tops, const Fan *fans, int j0, int j1, ViewEntry *views,
                         const LaunchState &state, hipStream_t st)
{
    const ViewShape sh = view_shape(s.n_b);
    const int threads = sh.n2 > 1 ? dev::kViewThreads
                                  : (int)std::min<int64_t>(dev::kViewThreads, std::max<int64_t>(256, ((int64_t)s.n_b + 63) / 64 * 64));
    hipLaunchKernelGGL(dev::k_views<Fan>, dim3((unsigned)((int64_t)(j1 - j0) * sh.n2)), dim3(threads), 0, st,
                       (const int32_t *)s.vorder, (const float4 *)s.pbox, tops, (const float4 *)s.gbox, (const int32_t *)s.voff, s.n_b, fans, j0,
                       views, state);
    if (sh.n3 > 1)
        hipLaunchKernelGGL(dev::k_view_blocks<Fan>, dim3((unsigned)((int64_t)(j1 - j0) * sh.n3)), dim3(64), 0, st,
                           (const float4 *)s.gbox, s.n_b, fans, j0, views);
}

}  // namespace sa
