// Persistent launches of the per-tile kernels (accrual, sampled,
// continuous shadow, contributions, adjoint).
//
// Their work is a list of units (64-point tile, part).  A part is a run of
// the launch's items (segments or instants): one output bin's run, every n-th
// item of it or of the launch, or all of them.  The tiles are cut into eight
// contiguous ranges, one per XCD (block b runs on XCD b mod 8), each with its
// own counter of units, all its tiles' first parts, then their second ones;
// a wave takes one unit per atomic from its XCD's range, then from the
// others'.  So the waves of an XCD walk neighbouring tiles on the same few
// segments' views, which its L2 holds, and stay resident until the work runs
// out: no SIMD idles behind a long tile, and a launch's tail is one unit
// long.  Dealing a run's items out in turn, instead of in consecutive pieces,
// gives every part its share of the low sun's long walks.  Tile by tile and
// in consecutive pieces before: contributions (5,000 prisms, 300k points) 1.27
// -> 1.07 ms, the sampled form (20,000 prisms, 1M points, 3 days) 5.43 -> 4.97
// ms, forward and adjoint at 1-minute knots (200k points) 12.4 -> 10.2 ms,
// the accrual form on the block scene 10.15 -> 10.04 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "sa_internal.h"
#include "traverse.h"

namespace sa {

constexpr int kSchedThreads = 256;               // threads per block of every persistent launch
constexpr int kSchedWaves = kSchedThreads / 64;  // waves per block
constexpr int kGrabStride = 32;                  // words between the eight counters (one 128-byte line each)

// Work of at most this many items (tiles x segments or chunks) per resident
// wave is dealt out, a unit per wave, instead of drawn from the counters: a
// draw is a round trip to memory, and a wave that finds nothing left has
// asked all eight counters.  (16,384 points and 64 prisms, a working day: 106
// -> 62 us; 40,000 points and 400 prisms after an edit: 252 -> 161 us; the
// sampled form on 20,000 points and 400 prisms: 167 -> 83 us.  More items a
// wave leave the lengths of the units uneven: at 4, 8 and 16 the sampled form
// on 60,000 points and 20,000 prisms takes 410, 307 and 306 us, contributions
// of 120,000 points 691, 710 and 710, the accrual form on 200,000 points 681,
// 680 and 699.)
constexpr int64_t kFewUnits = 8;

// Units per resident wave where a launch may cut its runs: one for every
// kChunkItems or kPieceItems items a wave has, between the bounds.  A unit has
// its set-up (its points, the roof test, of pieces a row of sums), and the last
// ones end one by one.  At 3, 4, 6, 8 and 16 units the accrual form on 200,000
// points (11 items a wave) takes 417, 440, 468, 470 and 515 us, on 400,000
// points (72 items) 739, 700, 703, 732 and 853; contributions of 300,000 points
// (29 items) 954, 827, 838, 874 and 943; at 4, 8, 16 and 24 forward and adjoint
// at 1-minute knots (280 and 370 items) 8.99, 7.50, 6.94 and 6.84 ms; at 8 and 24
// the sampled form on 1M points (300 chunks) 4.06 and 3.90 ms.
constexpr int64_t kChunkItems = 5, kPieceItems = 12;
constexpr int64_t kLeastChunks = 4, kLeastPieces = 3, kMostUnits = 24;

struct Sched {
    const int32_t *part_start;  // first item of each bin run of the launch (clipped to it), or null
    uint32_t *grab;             // eight counters, kGrabStride words apart, zero at launch; null: a
                                // unit per wave
    uint32_t n_tiles;
    uint32_t n_parts;
    int32_t strided;  // without part_start: part p takes items p, p + n_parts, ... (0: one part, every item)
    int32_t sub;    // with part_start: pieces each run is dealt into, item by item (0 or 1: whole runs)
};

namespace dev {

struct Unit {
    uint32_t tile;
    uint32_t part;
    int a, b;        // the unit's items a, a + step, ... below b
    int step;        // 1 but for strided parts
};

// The next unit of the launch whose Sched is parked at s_W, for items
// [a0, a1); false when none is left.  k counts the XCD ranges already
// drained (0 at the start).  Callers pass the unit's bounds through
// uniform(): set inside this loop, they would otherwise count as per-lane
// values and could not address scalar loads.
__device__ __forceinline__ bool next_unit(const lds_int *s_W, int a0, int a1, int &k, Unit &un)
{
    const Sched W = lds_uniform<Sched>(s_W);
    const int xcd = wg_id() & 7;
    for (; k < 8; ++k) {
        const int x = (xcd + k) & 7;
        const uint32_t lo = (uint32_t)((uint64_t)W.n_tiles * x >> 3);
        const uint32_t tiles = (uint32_t)((uint64_t)W.n_tiles * (x + 1) >> 3) - lo;
        uint32_t got = 0;
        if (W.grab) {
            if ((tid() & 63) == 0) got = atomicAdd(W.grab + kGrabStride * x, 1u);
            got = (uint32_t)__builtin_amdgcn_readlane((int)got, 0);
        } else {
            // a unit per wave: its own, then none
            got = (uint32_t)uniform((int)((wg_id() >> 3) * kSchedWaves + (tid() >> 6)));
            k = 7;
        }
        if (got < tiles * W.n_parts) {
            // the division runs on the vector unit: its result is made
            // scalar again for the scalar loads it addresses
            const uint32_t part = (uint32_t)uniform((int)(got / tiles));
            un.tile = lo + got - part * tiles;
            un.part = part;
            un.step = 1;
            if (W.part_start) {
                const uint32_t sub = W.sub > 1 ? (uint32_t)W.sub : 1u;
                const uint32_t run = part / sub, piece = part - run * sub;
                const int ra = max(ld((cint *)W.part_start + run), a0);
                const int rb = min(ld((cint *)W.part_start + run + 1), a1);
                un.a = ra + (int)piece;
                un.b = rb;
                un.step = (int)sub;
            } else if (W.strided) {
                un.a = a0 + (int)part;
                un.b = a1;
                un.step = (int)W.n_parts;
            } else {
                un.a = a0;
                un.b = a1;
            }
            k += W.grab ? 0 : 1;
            return true;
        }
    }
    return false;
}

}  // namespace dev

// How a persistent launch may cut a tile's items into parts.
enum class Split {
    kNone,        // one part per tile
    kUniqueBins,  // a part per bin run when no bin has two runs in the launch
                  // (each (tile, bin) is then one unit's: plain stores)
    kBinRuns,     // a part per bin run (outputs added atomically)
    kChunks,      // parts of every n-th item, enough units to keep every wave busy
                  // (outputs added atomically, or one per item)
    kRunPieces,   // as kUniqueBins, each run dealt into pieces, enough units to keep
                  // every wave busy (per-piece sums, added in a fixed order after)
};

// Blocks of a persistent launch of `kern`: the tuned count, else as many
// as the device holds at once.
template <class Kern>
static int64_t resident_blocks(Kern kern, const TileLaunch &L)
{
    if (L.grid_blocks > 0) return L.grid_blocks;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kSchedThreads, 0) != hipSuccess || per_cu < 1) {
        (void)hipGetLastError();
        per_cu = 1;
    }
    return (int64_t)per_cu * std::max(L.n_cu, 1);
}

// The units of a persistent launch over items [a0, a1) (segments or
// instants, whose bin runs are R) for `tiles` 64-point tiles; `blocks` is
// the launch size.
static inline Sched plan_units(const BinRuns &R, int a0, int a1, int64_t tiles, Split split, int64_t blocks,
                               uint32_t *grab, int64_t max_parts = 1)
{
    Sched W{nullptr, grab, (uint32_t)tiles, 1u, 0, 0};
    if (split == Split::kNone || a1 <= a0) return W;
    const int64_t waves = blocks * kSchedWaves;
    // the most parts that give every wave at most one unit (per XCD, whose
    // tiles are an eighth, rounded up)
    const int64_t single = (blocks / 8) * kSchedWaves / std::max<int64_t>((tiles + 7) / 8, 1);
    if (split == Split::kChunks) {
        const int64_t items = a1 - a0;
        const int64_t units = std::clamp(tiles * items / (waves * kChunkItems), kLeastChunks, kMostUnits);
        const int64_t want = std::max<int64_t>(1, (units * waves + tiles - 1) / tiles);
        int64_t parts = std::min(items, want);
        if (single >= 1 && tiles * items <= kFewUnits * waves) {
            parts = std::min(items, single);
            W.grab = nullptr;
        }
        while (parts > 1 && (uint64_t)tiles * (uint64_t)parts >= (1ull << 31)) parts /= 2;
        W.strided = 1;
        W.n_parts = (uint32_t)parts;
        return W;
    }
    if (R.dev == nullptr || R.start.size() < 2) return W;
    const auto &rs = R.start;
    const int r0 = (int)(std::upper_bound(rs.begin(), rs.end(), a0) - rs.begin()) - 1;
    const int r1 = (int)(std::upper_bound(rs.begin(), rs.end(), a1 - 1) - rs.begin()) - 1;
    if ((r1 <= r0 && split != Split::kRunPieces) || (uint64_t)tiles * (uint64_t)(r1 - r0 + 1) >= (1ull << 31))
        return W;
    if (split == Split::kUniqueBins || split == Split::kRunPieces) {
        std::vector<int32_t> bins(R.bin.begin() + r0, R.bin.begin() + r1 + 1);
        std::sort(bins.begin(), bins.end());
        if (std::adjacent_find(bins.begin(), bins.end()) != bins.end()) return W;
    }
    W.part_start = R.dev + r0;
    const int64_t runs = r1 - r0 + 1;
    W.n_parts = (uint32_t)runs;
    if (split == Split::kRunPieces) {
        // no piece shorter than one item, no more parts than the caller can hold
        int shortest = a1 - a0;
        for (int r = r0; r <= r1; ++r) shortest = std::min(shortest, std::min(rs[r + 1], a1) - std::max(rs[r], a0));
        const int64_t units = std::clamp(tiles * (a1 - a0) / (waves * kPieceItems), kLeastPieces, kMostUnits);
        const int64_t want = (units * waves + tiles * runs - 1) / (tiles * runs);
        int64_t sub = std::min<int64_t>(std::min<int64_t>(want, shortest), std::max<int64_t>(1, max_parts / runs));
        if (single >= runs && tiles * (a1 - a0) <= kFewUnits * waves) {
            sub = std::min(sub, single / runs);
            W.grab = nullptr;
        }
        while (sub > 1 && (uint64_t)tiles * (uint64_t)(runs * sub) >= (1ull << 31)) sub /= 2;
        if (sub > 1) {
            W.sub = (int32_t)sub;
            W.n_parts = (uint32_t)(runs * sub);
        }
    }
    return W;
}

// Blocks to launch: never more than the units need.
static inline int64_t unit_blocks(int64_t blocks, const Sched &W)
{
    if (!W.grab) return 8 * (((int64_t)(W.n_tiles + 7) / 8 * W.n_parts + kSchedWaves - 1) / kSchedWaves);
    const int64_t units = (int64_t)W.n_tiles * W.n_parts;
    return std::max<int64_t>(1, std::min<int64_t>(blocks, (units + kSchedWaves - 1) / kSchedWaves));
}

// Tiles of n points, refused beyond what the unit counters address.
static inline bool tile_count(int64_t n, int64_t &tiles, std::string &err)
{
    tiles = (n + 63) / 64;
    if (tiles >= (1ll << 31)) {
        err = "too many points";
        return false;
    }
    return true;
}

}  // namespace sa
