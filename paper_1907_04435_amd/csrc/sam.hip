// Gross shadow by raster shadow accrual maps (Sec. 4): per great-circle
// segment, a map of one depth slice per sample instant over a texel grid on
// a plane normal to the segment's start direction.  Step 1 fills every
// slice in one pass over (slice, prism) pairs: the depth at a texel is the
// largest distance along the light at which the ray from the texel centre
// toward the sun leaves a prism (its face nearest the sun).  Step 2 puts
// each point's shadow on every slice and counts the instants whose stored
// depth exceeds the point's own by more than the bias.  A map word holds an
// 8-bit segment stamp above a 24-bit depth (rounded down to a quantum of
// 1 / 2^24 of the segment's largest possible depth, about a millimetre for
// a city), so an integer maximum keeps the current segment's
// nearest-to-sun depth over any stale word, and the map is cleared only
// when it is allocated or after 255 segments.  Only texels that some point's
// shadow can fall on are built.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "sa_internal.h"

namespace sa {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / 64;

__global__ void k_sam_clear(uint32_t *p, int64_t n)
{
    const int64_t stride = (int64_t)n_wg() * wg_size();
    for (int64_t t = (int64_t)wg_id() * wg_size() + tid(); t < n; t += stride) p[t] = 0u;
}

// Bounds of the query points (x0, y0, z0, x1, y1, z1): of a block's share,
// then of all shares (one block).  Clamped to 1e9 so that a
// point at infinity leaves finite bounds.
constexpr int kBoundBlocks = 256;

__device__ __forceinline__ void block_bounds(float (&b)[6], float *out)
{
    __shared__ float red[kWavesPerBlock][6];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            const float v = __shfl_xor(b[c], o, 64);
            b[c] = c < 3 ? fminf(b[c], v) : fmaxf(b[c], v);
        }
    if ((tid() & 63) == 0)
#pragma unroll
        for (int c = 0; c < 6; ++c) red[tid() >> 6][c] = b[c];
    __syncthreads();
    if (tid() < 6) {
        float v = red[0][tid()];
        for (int w = 1; w < kWavesPerBlock; ++w) v = tid() < 3 ? fminf(v, red[w][tid()]) : fmaxf(v, red[w][tid()]);
        out[tid()] = fminf(fmaxf(v, -1e9f), 1e9f);
    }
}

__global__ __launch_bounds__(kThreads) void k_sam_bounds(const float *__restrict__ px, const float *__restrict__ py,
                                                         const float *__restrict__ pz, int64_t n, float *__restrict__ part)
{
    float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    const int64_t stride = (int64_t)n_wg() * kThreads;
    for (int64_t i = (int64_t)wg_id() * kThreads + tid(); i < n; i += stride) {
        const float x = px[i], y = py[i], z = pz[i];
        b[0] = fminf(b[0], x);
        b[1] = fminf(b[1], y);
        b[2] = fminf(b[2], z);
        b[3] = fmaxf(b[3], x);
        b[4] = fmaxf(b[4], y);
        b[5] = fmaxf(b[5], z);
    }
    block_bounds(b, part + 6 * wg_id());
}

__global__ __launch_bounds__(kThreads) void k_sam_bounds_all(const float *__restrict__ part, int blocks,
                                                             float *__restrict__ out)
{
    float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int t = tid(); t < blocks; t += kThreads)
#pragma unroll
        for (int c = 0; c < 6; ++c) b[c] = c < 3 ? fminf(b[c], part[6 * t + c]) : fmaxf(b[c], part[6 * t + c]);
    block_bounds(b, out);
}

// Range of the affine function c[0] x + c[1] y + c[2] z + c[3] over a box,
// widened by one and 2^-17 of its terms against rounding.
__device__ __forceinline__ void affine_range(const float (&c)[4], float x0, float y0, float z0, float x1, float y1,
                                             float z1, float &lo, float &hi)
{
    const float ax = c[0] * x0, bx = c[0] * x1, ay = c[1] * y0, by = c[1] * y1, az = c[2] * z0, bz = c[2] * z1;
    const float w = 1.f + 0x1p-17f * (fabsf(c[3]) + fmaxf(fabsf(ax), fabsf(bx)) + fmaxf(fabsf(ay), fabsf(by)) +
                                      fmaxf(fabsf(az), fabsf(bz)));
    lo = c[3] + fminf(ax, bx) + fminf(ay, by) + fminf(az, bz) - w;
    hi = c[3] + fmaxf(ax, bx) + fmaxf(ay, by) + fmaxf(az, bz) + w;
}

// Items of a wave's group: (slice, prism) pairs whose boxes are tested a lane
// each before the pairs left are built one by one.  Groups take prisms that
// lie n_b / per apart in hierarchy order, so neighbours (which the points see
// together) spread over the waves; larger groups leave too few waves when
// every prism is seen, as smaller ones do where there are few (30 slices of
// 300 prisms make 570 groups of 16: 500,000 points among them took 5.0 ms).
constexpr int kMostGroup = 16;
constexpr int64_t kLeastGroups = 16384;

// One wave per group, then per (slice, prism) of it whose shadow may fall on
// texels that points read: texels outside the box of all the points'
// shadows on the slice stay empty, for nothing reads them (1M points in the
// middle of a city of 20,000 prisms, a day at 1 minute, 2 m texels: 30.4 -> 3.0
// ms; where the points cover the city the tests cost nothing measurable).  The wave covers
// the texels of the prism's shadow on the plane (the box of its vertices'
// projections, clamped to the grid) in 8 x 8 tiles counted from the box's
// corner, those of them that meet the points' box, kTilesPerPass at a time in
// row order, each lane
// clipping the ray from its texel centre against the prism (height slab
// and every footprint edge's inner half-plane).  Within the box every
// clipping bound is an affine function of the texel's offset (i', j') from
// the box corner: the lanes first project one vertex each and form one
// edge's three coefficients each, then every pass reads an edge's
// coefficients from its lane and pays two FMAs and a min or max per texel.
// Depths are positive (the plane lies behind every prism) and quantised
// downward; with the segment's stamp above them a 32-bit integer maximum
// keeps the nearest-to-sun face of this segment.
constexpr int kTilesPerPass = 4;

__device__ __forceinline__ float wave_min(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

struct SamBuild {
    const float4 *verts;
    const int32_t *voff;
    const float *height;
    const float4 *pbox;
    const float *bounds;
    const SamSlice *slices;
    uint32_t *map;
    int32_t n_b, K;
    int32_t per;  // prisms per group
    uint32_t stamp;
    int32_t blocks;  // 0: nothing to build
    SamGrid g;
};

__device__ __forceinline__ void sam_build(const SamBuild &A, int block)
{
    const float4 *__restrict__ verts = A.verts;
    const int32_t *__restrict__ voff = A.voff;
    const float *__restrict__ height = A.height;
    const float4 *__restrict__ pbox = A.pbox;
    const float *__restrict__ bounds = A.bounds;
    const SamSlice *__restrict__ slices = A.slices;
    uint32_t *__restrict__ map = A.map;
    const int n_b = A.n_b, K = A.K;
    const uint32_t stamp = A.stamp;
    const SamGrid &g = A.g;
    const int lane = tid() & 63;
    const int lx = lane & 7, ly = lane >> 3;
    const uint32_t tag = stamp << 24;
    const int64_t T = (int64_t)g.nu * g.nv;
    const int per = A.per, groups = (n_b + per - 1) / per;  // per slice
    const int64_t nw = (int64_t)A.blocks * kWavesPerBlock;
    const int64_t w0 = (int64_t)block * kWavesPerBlock + __builtin_amdgcn_readfirstlane(tid() >> 6);
    for (int64_t it = w0; it < (int64_t)K * groups; it += nw) {
        const int k = (int)(it / groups);
        const int first = (int)(it - (int64_t)k * groups);
        const SamSlice s = slices[k];
        // grid coordinates (u, v) in texels of a point's shadow on the slice,
        // affine in the point (relative to o)
        const float du = s.dx * g.ux + s.dy * g.uy + s.dz * g.uz, dv = s.dx * g.vx + s.dy * g.vy + s.dz * g.vz;
        const float lu = du * s.inv_da, lv = dv * s.inv_da;
        const float cu[4] = {(g.ux - lu * g.ax) * g.inv_h, (g.uy - lu * g.ay) * g.inv_h, (g.uz - lu * g.az) * g.inv_h,
                             (lu * g.c - g.u0) * g.inv_h};
        const float cv[4] = {(g.vx - lv * g.ax) * g.inv_h, (g.vy - lv * g.ay) * g.inv_h, (g.vz - lv * g.az) * g.inv_h,
                             (lv * g.c - g.v0) * g.inv_h};
        // the box of the points' shadows in texels, empty at ri1 < ri0
        float ri0, ri1, rj0, rj1;
        affine_range(cu, bounds[0] - g.ox, bounds[1] - g.oy, bounds[2] - g.oz, bounds[3] - g.ox, bounds[4] - g.oy,
                     bounds[5] - g.oz, ri0, ri1);
        affine_range(cv, bounds[0] - g.ox, bounds[1] - g.oy, bounds[2] - g.oz, bounds[3] - g.ox, bounds[4] - g.oy,
                     bounds[5] - g.oz, rj0, rj1);
        ri0 = fminf(fmaxf(floorf(ri0), 0.f), (float)g.nu);
        ri1 = fmaxf(fminf(floorf(ri1), (float)(g.nu - 1)), -1.f);
        rj0 = fminf(fmaxf(floorf(rj0), 0.f), (float)g.nv);
        rj1 = fmaxf(fminf(floorf(rj1), (float)(g.nv - 1)), -1.f);
        bool meets = false;
        const int mine = first + lane * groups;
        if (lane < per && mine < n_b) {
            const float4 q = pbox[mine];
            float bu0, bu1, bv0, bv1;
            affine_range(cu, q.x - g.ox, q.y - g.oy, -g.oz, q.z - g.ox, q.w - g.oy, height[mine] - g.oz, bu0, bu1);
            affine_range(cv, q.x - g.ox, q.y - g.oy, -g.oz, q.z - g.ox, q.w - g.oy, height[mine] - g.oz, bv0, bv1);
            meets = bu1 >= ri0 && bu0 <= ri1 + 1.f && bv1 >= rj0 && bv0 <= rj1 + 1.f;
        }
        for (uint64_t left = __ballot(meets); left; left &= left - 1) {
            const int b = first + (int)__builtin_ctzll(left) * groups;
            const int e0 = voff[b], ne = voff[b + 1] - e0;
            const float H = height[b];
            const float zlo = -g.oz, zhi = H - g.oz;
            // the prism's shadow: hull of its 2 x ne vertices' projections, a
            // vertex per lane
            float umin = INFINITY, umax = -INFINITY, vmin = INFINITY, vmax = -INFINITY;
            for (int c = 0; c < ne; c += 64) {
                if (c + lane < ne) {
                    const float4 q = verts[e0 + c + lane];
                    const float rx = q.x - g.ox, ry = q.y - g.oy;
#pragma unroll
                    for (int top = 0; top < 2; ++top) {
                        const float rz = top ? zhi : zlo;
                        const float lam = (rx * g.ax + ry * g.ay + rz * g.az - g.c) * s.inv_da;
                        const float px = rx - lam * s.dx, py = ry - lam * s.dy, pz = rz - lam * s.dz;
                        const float pu = px * g.ux + py * g.uy + pz * g.uz;
                        const float pv = px * g.vx + py * g.vy + pz * g.vz;
                        umin = fminf(umin, pu);
                        umax = fmaxf(umax, pu);
                        vmin = fminf(vmin, pv);
                        vmax = fmaxf(vmax, pv);
                    }
                }
            }
            umin = wave_min(umin);
            umax = wave_max(umax);
            vmin = wave_min(vmin);
            vmax = wave_max(vmax);
            // a centimetre of slack against the rounding of the projections;
            // clamped in float before the conversion to integers
            const float fi0 = fmaxf(floorf((umin - 0.01f - g.u0) * g.inv_h), 0.f);
            const float fi1 = fminf(floorf((umax + 0.01f - g.u0) * g.inv_h), (float)(g.nu - 1));
            const float fj0 = fmaxf(floorf((vmin - 0.01f - g.v0) * g.inv_h), 0.f);
            const float fj1 = fminf(floorf((vmax + 0.01f - g.v0) * g.inv_h), (float)(g.nv - 1));
            if (!(fi0 <= fi1 && fj0 <= fj1)) continue;
            const int i0 = __builtin_amdgcn_readfirstlane((int)fi0), j0 = __builtin_amdgcn_readfirstlane((int)fj0);
            const int W = __builtin_amdgcn_readfirstlane((int)fi1) - i0 + 1;
            const int Hh = __builtin_amdgcn_readfirstlane((int)fj1) - j0 + 1;
            // of its tiles, those that meet the points' box
            const int ta = max((int)ri0 - i0, 0) >> 3, tb = min((int)ri1 - i0, W - 1) >> 3;
            const int va = max((int)rj0 - j0, 0) >> 3, vb = min((int)rj1 - j0, Hh - 1) >> 3;
            if ((int)ri1 < i0 || (int)rj1 < j0 || ta > tb || va > vb) continue;
            const int tx0 = __builtin_amdgcn_readfirstlane(ta), ty0 = __builtin_amdgcn_readfirstlane(va);
            const int tx_n = __builtin_amdgcn_readfirstlane(tb) - tx0 + 1;
            const int ty_n = __builtin_amdgcn_readfirstlane(vb) - ty0 + 1;
            uint32_t *slice = map + (int64_t)k * T;
            // the ray from the centre of texel (i0 + i', j0 + j'):
            // X0 + i' h u + j' h v + lam d
            const float cu0 = g.u0 + ((float)i0 + 0.5f) * g.h, cv0 = g.v0 + ((float)j0 + 0.5f) * g.h;
            const float X0 = g.c * g.ax + cu0 * g.ux + cv0 * g.vx;
            const float Y0 = g.c * g.ay + cu0 * g.uy + cv0 * g.vy;
            const float Z0 = g.c * g.az + cu0 * g.uz + cv0 * g.vz;
            // height slab: lam in [(zlo - Z) / dz, (zhi - Z) / dz]; the sun is
            // above the horizon (dz > 0)
            const float inv_dz = 1.f / s.dz;
            const float zl0 = (zlo - Z0) * inv_dz, zh0 = (zhi - Z0) * inv_dz;
            const float zi = -g.h * g.uz * inv_dz, zj = -g.h * g.vz * inv_dz;
            const int n_tiles = tx_n * ty_n;
            const float fi = (float)lx, fj = (float)ly;
            const float zl = fmaf(zj, fj, fmaf(zi, fi, zl0)), zh = fmaf(zj, fj, fmaf(zi, fi, zh0));
            // edge c + lane: along the ray its inner-side function is
            // f0 + fu i' + fv j' + lam gd (n.(x - p0) with n the outward normal;
            // inside where <= 0).  kind 1: gd > 0, the crossing
            // lam = A + B i' + C j' bounds lam from above; kind -1: from below;
            // kind 0: parallel, (A, B, C) = (f0, fu, fv) must stay <= 0.
            auto edge_coef = [&](int c, float &eA, float &eB, float &eC, int &kind) {
                eA = eB = eC = 0.f;
                kind = 0;
                if (c + lane < ne) {
                    const float4 q = verts[e0 + c + lane];
                    const float f0 = q.z * (X0 - (q.x - g.ox)) + q.w * (Y0 - (q.y - g.oy));
                    const float fu = g.h * (q.z * g.ux + q.w * g.uy), fv = g.h * (q.z * g.vx + q.w * g.vy);
                    const float gd = q.z * s.dx + q.w * s.dy;
                    if (gd != 0.f) {
                        const float rg = -1.f / gd;
                        eA = f0 * rg;
                        eB = fu * rg;
                        eC = fv * rg;
                        kind = gd > 0.f ? 1 : -1;
                    } else {
                        eA = f0;
                        eB = fu;
                        eC = fv;
                    }
                }
            };
            float eA0, eB0, eC0;
            int kind0;
            edge_coef(0, eA0, eB0, eC0, kind0);  // the first 64 edges, once per (slice, prism)
            for (int t0 = 0; t0 < n_tiles; t0 += kTilesPerPass) {
                // the pass's tiles in row order: offsets (in texels) of each
                // tile's corner, the same for every lane
                float ox[kTilesPerPass], oy[kTilesPerPass];
                int tx = t0 % tx_n, ty = t0 / tx_n;
#pragma unroll
                for (int r = 0; r < kTilesPerPass; ++r) {
                    ox[r] = (float)(8 * (tx0 + tx));
                    oy[r] = (float)(8 * (ty0 + ty));
                    if (++tx == tx_n) {
                        tx = 0;
                        ++ty;
                    }
                }
                float lo[kTilesPerPass], hi[kTilesPerPass];
#pragma unroll
                for (int r = 0; r < kTilesPerPass; ++r) {
                    lo[r] = fmaxf(0.f, fmaf(zj, oy[r], fmaf(zi, ox[r], zl)));
                    hi[r] = fmaf(zj, oy[r], fmaf(zi, ox[r], zh));
                }
                for (int c = 0; c < ne; c += 64) {
                    float eA = eA0, eB = eB0, eC = eC0;
                    int kind = kind0;
                    if (c > 0) edge_coef(c, eA, eB, eC, kind);  // footprints beyond 64 vertices
                    const int m_n = min(64, ne - c);
                    for (int m = 0; m < m_n; ++m) {
                        const float A = lane_value(eA, m), B = lane_value(eB, m), Cv = lane_value(eC, m);
                        const int kd = __builtin_amdgcn_readlane(kind, m);
                        const float base = fmaf(B, fi, fmaf(Cv, fj, A));
                        if (kd > 0) {
#pragma unroll
                            for (int r = 0; r < kTilesPerPass; ++r)
                                hi[r] = fminf(hi[r], fmaf(Cv, oy[r], fmaf(B, ox[r], base)));
                        } else if (kd < 0) {
#pragma unroll
                            for (int r = 0; r < kTilesPerPass; ++r)
                                lo[r] = fmaxf(lo[r], fmaf(Cv, oy[r], fmaf(B, ox[r], base)));
                        } else {
                            // parallel to the edge: outside it, no hit
#pragma unroll
                            for (int r = 0; r < kTilesPerPass; ++r)
                                if (fmaf(Cv, oy[r], fmaf(B, ox[r], base)) > 0.f) lo[r] = INFINITY;
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < kTilesPerPass; ++r) {
                    const int ii = (int)ox[r] + lx, jj = (int)oy[r] + ly;
                    if (t0 + r < n_tiles && ii < W && jj < Hh && lo[r] <= hi[r])
                        atomicMax(slice + (int64_t)(j0 + jj) * g.nu + (i0 + ii),
                                  tag | (uint32_t)fminf(hi[r] * g.inv_dq, 16777215.f));
                }
            }
        }
    }
}

// One thread per point: its shadow on each slice, the stored depth there
// (if written for this segment) against its own depth plus the bias; the
// segment's counts and minutes added to the point's bin.
struct SamQuery {
    const float *px, *py, *pz;
    const SamSlice *slices;
    const uint32_t *map;
    int32_t *counts;
    float *minutes;
    int64_t n;
    float scale;
    int32_t K, bin;
    uint32_t stamp;
    int32_t blocks;  // 0: nothing to ask
    SamGrid g;
};

__device__ __forceinline__ void sam_query(const SamQuery &A, int block)
{
    const float *__restrict__ px = A.px, *__restrict__ py = A.py, *__restrict__ pz = A.pz;
    const SamSlice *__restrict__ slices = A.slices;
    const uint32_t *__restrict__ map = A.map;
    int32_t *__restrict__ counts = A.counts;
    float *__restrict__ minutes = A.minutes;
    const int64_t n = A.n;
    const float scale = A.scale;
    const int K = A.K, bin = A.bin;
    const uint32_t stamp = A.stamp;
    const SamGrid &g = A.g;
    const int64_t T = (int64_t)g.nu * g.nv;
    const int64_t stride = (int64_t)A.blocks * kThreads;
    for (int64_t i = (int64_t)block * kThreads + tid(); i < n; i += stride) {
        const float rx = px[i] - g.ox, ry = py[i] - g.oy, rz = pz[i] - g.oz;
        const float ra = rx * g.ax + ry * g.ay + rz * g.az - g.c;
        int cnt = 0;
        float mins = 0.f;
        for (int k = 0; k < K; ++k) {
            const SamSlice s = slices[k];
            const float lam = ra * s.inv_da;
            const float qx = rx - lam * s.dx, qy = ry - lam * s.dy, qz = rz - lam * s.dz;
            const float fu = floorf((qx * g.ux + qy * g.uy + qz * g.uz - g.u0) * g.inv_h);
            const float fv = floorf((qx * g.vx + qy * g.vy + qz * g.vz - g.v0) * g.inv_h);
            if (fu >= 0.f && fu < (float)g.nu && fv >= 0.f && fv < (float)g.nv) {
                // a word of an earlier segment (another stamp) is empty here
                const uint32_t m = map[(int64_t)k * T + (int64_t)fv * g.nu + (int64_t)fu];
                if ((m >> 24) == stamp && (float)(m & 0xffffffu) * g.dq > lam + g.bias) {
                    ++cnt;
                    mins += s.w;
                }
            }
        }
        if (counts) counts[(int64_t)bin * n + i] += cnt;
        if (minutes) minutes[(int64_t)bin * n + i] += mins * scale;
    }
}

// One segment's map is built while the one before is asked, in one launch with
// the blocks of both in even mixture: the build computes (60 % of VALU issue),
// the query waits for its map words, and on few points or prisms neither fills
// the device.  One after the other: 60,000 points among 300 prisms at 1.5 m 3.26
// -> 1.54 ms (with groups as large as they may be), among 5,000 2.98 -> 2.22, 5,000
// points 1.66 -> 1.03; 1M points among 20,000 at 2 m, which fill it, 4.90 -> 5.01.
// At 5 waves per SIMD (84 VGPRs) that is 5.38, at 7 and 8 (spilling) 5.23 and 5.60.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_sam_step(SamBuild B, SamQuery Q)
{
    const uint32_t total = (uint32_t)(B.blocks + Q.blocks), b = (uint32_t)wg_id();
    const uint32_t q0 = (uint32_t)((uint64_t)b * Q.blocks / total), q1 = (uint32_t)((uint64_t)(b + 1) * Q.blocks / total);
    if (q1 > q0)
        sam_query(Q, (int)q0);
    else
        sam_build(B, (int)(b - q0));
}

// Plane and grid of one segment, FP64 (the float32 copy is relative to o):
// normal a; u = z x a normalised (east at the zenith), v = a x u; the plane
// 1 m behind the box corner farthest from the sun; the grid covers the
// box's projections along a and b (those along every direction between them
// lie in between) with a texel of margin.
bool sam_grid(const double box[6], const double *a, const double *b, double h, double bias, SamGrid &g)
{
    double u[3] = {-a[1], a[0], 0.0};
    const double ul = std::sqrt(u[0] * u[0] + u[1] * u[1]);
    if (ul > 1e-9) {
        u[0] /= ul;
        u[1] /= ul;
    } else {
        u[0] = 1.0;
        u[1] = 0.0;
    }
    const double v[3] = {a[1] * u[2] - a[2] * u[1], a[2] * u[0] - a[0] * u[2], a[0] * u[1] - a[1] * u[0]};
    double c = INFINITY;
    double X[8][3];
    for (int q = 0; q < 8; ++q) {
        X[q][0] = box[(q & 4) ? 3 : 0];
        X[q][1] = box[(q & 2) ? 4 : 1];
        X[q][2] = box[(q & 1) ? 5 : 2];
        c = std::min(c, X[q][0] * a[0] + X[q][1] * a[1] + X[q][2] * a[2]);
    }
    c -= 1.0;
    double umin = INFINITY, umax = -INFINITY, vmin = INFINITY, vmax = -INFINITY;
    for (const double *d : {a, b}) {
        const double da = d[0] * a[0] + d[1] * a[1] + d[2] * a[2];
        for (int q = 0; q < 8; ++q) {
            const double lam = (X[q][0] * a[0] + X[q][1] * a[1] + X[q][2] * a[2] - c) / da;
            const double p[3] = {X[q][0] - lam * d[0], X[q][1] - lam * d[1], X[q][2] - lam * d[2]};
            const double pu = p[0] * u[0] + p[1] * u[1] + p[2] * u[2];
            const double pv = p[0] * v[0] + p[1] * v[1] + p[2] * v[2];
            umin = std::min(umin, pu);
            umax = std::max(umax, pu);
            vmin = std::min(vmin, pv);
            vmax = std::max(vmax, pv);
        }
    }
    const double u0 = std::floor(umin / h) * h - h, v0 = std::floor(vmin / h) * h - h;
    const double nu = std::ceil((umax - u0) / h) + 1.0, nv = std::ceil((vmax - v0) / h) + 1.0;
    if (!(nu >= 1.0 && nv >= 1.0 && nu < 2e9 && nv < 2e9)) return false;
    const double o[3] = {0.5 * (box[0] + box[3]), 0.5 * (box[1] + box[4]), 0.5 * (box[2] + box[5])};
    g.ax = (float)a[0];
    g.ay = (float)a[1];
    g.az = (float)a[2];
    g.ux = (float)u[0];
    g.uy = (float)u[1];
    g.uz = (float)u[2];
    g.vx = (float)v[0];
    g.vy = (float)v[1];
    g.vz = (float)v[2];
    g.c = (float)(c - (o[0] * a[0] + o[1] * a[1] + o[2] * a[2]));
    g.u0 = (float)(u0 - (o[0] * u[0] + o[1] * u[1] + o[2] * u[2]));
    g.v0 = (float)(v0 - (o[0] * v[0] + o[1] * v[1] + o[2] * v[2]));
    g.h = (float)h;
    g.inv_h = (float)(1.0 / h);
    g.nu = (int32_t)nu;
    g.nv = (int32_t)nv;
    g.ox = (float)o[0];
    g.oy = (float)o[1];
    g.oz = (float)o[2];
    g.bias = (float)bias;
    // every slice direction d lies on the arc from a to b, so d.a >= a.b and
    // no depth exceeds (max corner.a - c) / (a.b); 1 % of slack
    double cmax = -INFINITY;
    for (int q = 0; q < 8; ++q) cmax = std::max(cmax, X[q][0] * a[0] + X[q][1] * a[1] + X[q][2] * a[2]);
    const double ab = a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
    if (!(ab > 0.0)) return false;
    const double lam_max = 1.01 * (cmax - c) / ab;
    g.dq = (float)(lam_max / 16777215.0);
    g.inv_dq = (float)(16777215.0 / lam_max);
    return true;
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

sa_status launch_sam(const DeviceScene &s, const DevicePath &p, const PointsView &pts, double texel,
                     double bias, const double box[6], int64_t max_texels, bool cap_both, float scale, int32_t *counts,
                     float *minutes, Scratch &scr, uint32_t &stamp, hipStream_t st, std::string &err)
{
    if (s.n_b == 0 || pts.n == 0 || p.n_samples == 0) return SA_OK;
    if (!p.sam_slices || p.seg_host.size() != (size_t)p.n_segs) {
        err = "sa_sam_accumulate: path has no raster slices";
        return SA_ERR_INVALID_ARG;
    }
    // every segment's grid first: the map buffer is sized for the largest
    std::vector<SamGrid> grids(p.seg_host.size());
    int64_t most = 0;
    for (size_t j = 0; j < p.seg_host.size(); ++j) {
        const SamSegHost &sh = p.seg_host[j];
        if (sh.ns == 0) continue;
        if (!sam_grid(box, sh.a, sh.b, texel, bias, grids[j])) {
            err = "sa_sam_accumulate: texel grid out of range";
            return SA_ERR_CAPACITY;
        }
        // in floating point first: nu * nv * ns may not fit 64 bits
        const double texels = (double)grids[j].nu * (double)grids[j].nv * (double)sh.ns;
        if (texels > (double)max_texels) {
            err = "sa_sam_accumulate: a segment's map needs " + std::to_string(texels) +
                  " texels, above the cap (larger texels, or a higher cap)";
            return SA_ERR_CAPACITY;
        }
        most = std::max(most, (int64_t)grids[j].nu * grids[j].nv * sh.ns);
    }
    // the points' bounds and their shares lie behind the map
    // two maps, one built while the other is asked; one where both cannot be had
    // or would pass the caller's cap (one takes 9.0 ms, where two take 8.2: 2M
    // points in the block scene, maps of 1.3e9 texels)
    const size_t map_bytes = ((size_t)most * sizeof(uint32_t) + 255) & ~(size_t)255;
    const size_t bound_bytes = 6 * (kBoundBlocks + 1) * sizeof(float);
    const size_t one = map_bytes + bound_bytes, need = one + map_bytes;
    auto clear_all = [&]() {
        const int64_t words = (int64_t)((scr.bytes - bound_bytes) / sizeof(uint32_t));
        hipLaunchKernelGGL(k_sam_clear, dim3((unsigned)std::min<int64_t>((words + kThreads - 1) / kThreads, 65536)),
                           dim3(kThreads), 0, st, (uint32_t *)scr.ptr, words);
        stamp = 0;
    };
    const uint32_t made = scr.made;
    const bool wish = !cap_both || most <= max_texels / 2;
    if (!(wish && reserve_wish(scr, need, st)) && !reserve(scr, one, st)) {
        err = "no room for a raster map (under stream capture an eager call of the size comes first)";
        return SA_ERR_OOM;
    }
    if (scr.made != made) {
        clear_all();
        SA_CHECK_LAUNCH("raster map clear");
    }
    const bool two = scr.bytes >= need;
    uint32_t *maps[2] = {(uint32_t *)scr.ptr, (uint32_t *)((char *)scr.ptr + (two ? map_bytes : 0))};
    float *bounds = (float *)((char *)scr.ptr + scr.bytes - bound_bytes);
    const unsigned bblocks = (unsigned)std::min<int64_t>((pts.n + kThreads - 1) / kThreads, kBoundBlocks);
    hipLaunchKernelGGL(k_sam_bounds, dim3(bblocks), dim3(kThreads), 0, st, pts.x, pts.y, pts.z, pts.n, bounds + 6);
    hipLaunchKernelGGL(k_sam_bounds_all, dim3(1), dim3(kThreads), 0, st, (const float *)(bounds + 6), (int)bblocks,
                       bounds);
    SA_CHECK_LAUNCH("raster point bounds");
    const unsigned qblocks = (unsigned)std::min<int64_t>((pts.n + kThreads - 1) / kThreads, 16384);
    SamBuild B{};
    SamQuery Q{};
    auto step = [&]() {
        if (B.blocks + Q.blocks > 0)
            hipLaunchKernelGGL(k_sam_step, dim3((unsigned)(B.blocks + Q.blocks)), dim3(kThreads), 0, st, B, Q);
        B.blocks = Q.blocks = 0;
    };
    int turn = 0;
    for (size_t j = 0; j < p.seg_host.size(); ++j) {
        const SamSegHost &sh = p.seg_host[j];
        if (sh.ns == 0) continue;
        const SamGrid &g = grids[j];
        const SamSlice *sl = p.sam_slices + sh.first;
        if (stamp >= 255u) {
            step();  // the last map is asked before it is cleared
            clear_all();
            SA_CHECK_LAUNCH("raster map clear");
        }
        ++stamp;
        int per = kMostGroup;
        while (per > 1 && (int64_t)sh.ns * ((s.n_b + per - 1) / per) < kLeastGroups) per /= 2;
        const int64_t items = (int64_t)sh.ns * ((s.n_b + per - 1) / per);
        uint32_t *map = maps[turn ^= 1];
        B = SamBuild{s.verts, s.voff, s.height, s.pbox, bounds, sl, map, s.n_b, sh.ns, per, stamp,
                     (int32_t)std::min<int64_t>((items + kWavesPerBlock - 1) / kWavesPerBlock, 32768), g};
        if (!two && Q.blocks > 0) {  // the one map is asked before it is built again
            const SamBuild next = B;
            B.blocks = 0;
            step();
            B = next;
        }
        step();
        SA_CHECK_LAUNCH("raster map");
        Q = SamQuery{pts.x, pts.y, pts.z, sl, map, counts, minutes, pts.n, scale, sh.ns, sh.bin, stamp, (int32_t)qblocks, g};
    }
    step();
    SA_CHECK_LAUNCH("raster map query");
    return SA_OK;
}

}  // namespace sa
