// indexer_plan.h -- host-side planning of the indexer's grid. Plain C++ with
// no HIP dependency, so the library and a sanitizer build on the CPU compile
// the same code.
#ifndef GVR_INDEXER_PLAN_H
#define GVR_INDEXER_PLAN_H

#include <stdint.h>

#include <algorithm>

namespace gvr_idx {

constexpr int kTile = 32;                // keys per ring slot (two 16-key matrix steps)
constexpr int kTilesPerWave = 32;        // ring slots of one wave's run (1024 keys)
constexpr int kMinRun = 8 * kTile;       // shortest wave run the grid sizing picks (256 keys)
constexpr int kSharedPerCu = 3;          // workgroups per compute unit whose waves share key tiles (D = 128)
constexpr int kSpread = 32;              // consecutive workgroups go to 8 XCDs in turn, in each to 4 shader engines

// Keys per wave run when the grid is cut for m workgroups on each of `cus`
// compute units (slots = m * cus), wpr waves side by side, and the share of
// those places that the grid fills.
struct Cut {
    int run;
    double fill;
    int64_t rounds, chunks;
};
inline Cut cut_for(int64_t ld, int64_t caches, int wpr, int64_t slots) {
    const int64_t natural = (int64_t)wpr * kTilesPerWave * kTile;
    const int64_t nat = (ld + natural - 1) / natural;
    const int64_t rounds = std::max<int64_t>(1, nat * caches / slots);
    const int64_t chunks = std::max<int64_t>(1, rounds * slots / caches);
    const int64_t per = (ld + chunks - 1) / chunks;                          // keys per chunk
    const int64_t r = ((per + wpr - 1) / wpr + kTile - 1) / kTile * kTile;   // per wave, whole tiles
    // At most three natural runs (chunks >= nat / 3 above); the bound keeps a
    // run's bytes far inside the 32-bit range of its buffer resource.
    const int run = (int)std::max<int64_t>(std::min<int64_t>(r, 4 * kTilesPerWave * kTile), kMinRun);
    const int64_t got = (ld + (int64_t)wpr * run - 1) / ((int64_t)wpr * run);
    return {run, (double)(got * caches) / ((double)rounds * (double)slots), rounds, got};
}

struct Grid {
    int run;        // keys per wave run
    bool limited;   // unused LDS keeps at most kSharedPerCu workgroups on a compute unit
    int64_t places;   // workgroups of one round the grid is cut for (0: unknown)
};

// Key chunks per cache. The natural size gives every wave a run of
// kTilesPerWave tiles; the grid is then resized to whole rounds of m
// workgroups per compute unit: one round when the natural grid fits (small
// batches get finer chunks that reach more compute units, runs of at least
// kMinRun keys), else as many full rounds as it fills (no partly filled last
// round). m is the smallest from 2 on that the caches fill to nine tenths,
// else the best filled one: fewer workgroups with longer runs pay the queries
// and the first loads less often, and places left empty cost more than that.
// 40 x 1 rows of 20000 keys (H = 64, D = 128): 18.7 us at m = 2, 20.9 at 3,
// 21.3 at 4; 100 x 1 of 30000 50.9 / 57.1 / 57.2; 300 x 1 of 3000, where
// m = 2 is 59 % full, 29.6 / 25.8 / 23.0. It is not the best m everywhere:
// 8 x 1 of 131072 takes 25.7 us where m = 3 takes 24.1, 16 x 1 ragged of
// 70000 22.8 where m = 4 takes 20.6, 40 x 4 ragged of 20000 (H = 32) 32.6
// where m = 3 takes 30.1; the places are counted from the stride, so ragged
// rows fill fewer of them.
//
// Where a cache's rows do not pair (groups of three, and H = 128; `shared`),
// several waves read each key tile, and the reuse is the L1's. With D = 128
// more than three such workgroups per compute unit evict each other's tiles,
// so the grid is cut for three and unused LDS keeps it there (64 x 3 ragged
// rows of 60000 keys, H = 32: 135.9 us against 140.7 at four and 147.0
// unlimited). One round of two or more chunks per cache that leaves a tenth of
// those places empty takes a larger m that fills better, without the limit
// (200 x 3 of 6000, H = 32: 72.6 us in 78 % of three, 57.7 in 98 % of four;
// H = 64 76.6 and 60.1); with one chunk per cache, or in more rounds, the
// limit pays all the same (500 x 3 of 1500, H = 32: 36.4 us in 65 % of three,
// 40.7 in 98 % of four; 400 x 3 of 6000 112 in 87 %, 125). With D = 64 every
// resident workgroup counts (40 x 3 of 20000, H = 64: 26.5 against 32.5 at
// m = 2).
inline Grid plan_grid(int64_t ld, int64_t caches, int wpr, int per_cu, int cus, bool shared, int D) {
    const bool limit = shared && D == 128;
    Grid g{kTilesPerWave * kTile, limit, 0};
    if (per_cu <= 0) return g;   // residency unknown: the natural size
    double best = -1.0;
    int m = std::min(2, per_cu);
    if (shared) m = limit ? std::min(kSharedPerCu, per_cu) : per_cu;
    for (; m <= per_cu && best < 0.9; ++m) {
        const Cut c = cut_for(ld, caches, wpr, (int64_t)m * cus);
        if (c.fill > best) {
            best = c.fill;
            g = Grid{c.run, limit && m <= kSharedPerCu, (int64_t)m * cus};
        }
        if (g.limited && (c.rounds > 1 || c.chunks == 1)) break;
    }
    return g;
}

// Workgroup b serves cache g = b / chunks and its chunk (b % chunks +
// first_chunk(g)) % chunks. Where rows differ in length their last chunks hold
// no keys, and with a chunk count that is a multiple of 8, which whole rounds
// of 256 m places make common, a chunk would meet the same XCD in every cache
// (of 16 and 32, the same shader engine too): the others would idle. Caches
// that would meet the same places therefore start at chunks spread evenly over
// the cache. Ragged rows of up to 33000 keys: 400 x 3 (H = 32, D = 64) 336 ->
// 221 us, 256 x 4 (H = 32, D = 128) 281 -> 214, 300 x 1 (H = 64, D = 128)
// 217 -> 187; equal lengths as before. A grid of one round has no place
// waiting for another's chunks, and starting elsewhere costs locality (equal
// lengths, H = 32, D = 128, 64 x 3 of 25000 in two rounds, where tiles are
// shared: 77.8 -> 84.3 us), so it is done from two rounds on, from three where
// tiles are shared. Other chunk counts spread by
// themselves (300 x 3 ragged of 16384, D = 64, 12 chunks: 100.5 us, 124.6
// rotated).
struct Rotation {
    int shift, mask, step;   // first_chunk(g) = ((g >> shift) & mask) * step
};
inline Rotation rotation(const Grid& g, int64_t chunks, int64_t caches, bool ragged) {
    if (!ragged || chunks % 8 != 0) return {0, 0, 0};
    if (2 * chunks * caches < (g.limited ? 5 : 3) * g.places) return {0, 0, 0};   // (rounds to the nearest)
    int common = 8, shift = 2;   // places that consecutive caches share: kSpread >> shift
    while (common < kSpread && chunks % (2 * common) == 0) {
        common *= 2;
        --shift;
    }
    return {shift, common - 1, (int)(chunks / common)};
}
inline int first_chunk(int g, int shift, int mask, int step) { return ((g >> shift) & mask) * step; }

}  // namespace gvr_idx

#endif  // GVR_INDEXER_PLAN_H
