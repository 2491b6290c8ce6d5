// guess.h -- Phase 1 of Guess-Verify-Refine (Sec. 4.2.1) over the scores at
// a strided sample of the previous step's Top-K, as one wave computes it.
// Shared by the Top-K kernel (which gathers the sampled scores itself) and
// the indexer kernel (which scores the sampled keys while it computes the
// row, for gvr_indexer_topk), so both give the same T_spec bit for bit.
#ifndef GVR_GUESS_H
#define GVR_GUESS_H

#include "wave_ops.h"

namespace gvr_dev {

constexpr int kGuessSamples = 256;   // guessed indices used: every st-th entry of prev_topk, st = ceil(K / 256)
constexpr int kGuessBins = 1024;     // bins over the sampled keys' range
constexpr int kSpecQuantile = 65;    // T_spec: sampled key of rank ceil(65 / 2048 * samples) from the bottom
constexpr int kGuessMaxK = 2048;     // the quantile's denominator (the largest K)

// Sample stride and sample count for a Top-K of size K.
__host__ DEV int guess_stride(int K) { return (K + kGuessSamples - 1) / kGuessSamples; }
__host__ DEV int guess_count(int K) {
    const int st = guess_stride(K);
    return (K + st - 1) / st;
}

// The statistics of one row's sample: T_spec (0xFFFFFFFF without a valid
// sample), the number of valid samples, their smallest and largest key, and
// the sum of their values (for pmean; summed in a fixed order).
struct GuessStats {
    uint32_t ts;
    int cnt;
    uint32_t mn, mx;
    float sum;
};

// Words of a row's GuessStats as gvr_indexer_topk hands them to the Top-K.
constexpr int kGuessWords = 8;

// One wave: lane l holds samples l + 64 c (c < 4), value gv[c], valid ok[c].
// T_spec is the lower edge of the bin (kGuessBins bins over [pmin, pmax])
// holding the valid sample of rank ceil(65 m / 2048) from the bottom (m valid
// samples), at least key 1. The row waits for this one wave, whose time is
// its dependent instructions: the rank's bin comes from a binary search over
// the bin's bits with ballots (every sample stays in its register), not from
// a histogram in LDS, and the sum is formed only if `want_sum`. From the
// sampled scores' arrival to T_spec published: 1.28 -> 0.85 us for one 8K row.
DEV GuessStats guess_from_samples(const float (&gv)[4], const bool (&ok)[4], bool want_sum) {
    uint32_t gk[4];
    int cnt = 0;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        gk[c] = key_of(gv[c]);
        mn = min(mn, ok[c] ? gk[c] : 0xFFFFFFFFu);
        mx = max(mx, ok[c] ? gk[c] : 0u);
        cnt += (int)__popcll(__ballot(ok[c]));
    }
    mn = wave_min_u(mn);
    mx = wave_max_u(mx);
    float sum = 0.f;
    if (want_sum) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (ok[c]) sum += gv[c];
        sum = wave_sum_f(sum);
    }
    uint32_t ts = 0xFFFFFFFFu;
    if (cnt > 0) {
        const uint64_t width = (uint64_t)mx - mn + 1;
        const uint32_t sh = bin_shift(width, log2i(kGuessBins));
        uint32_t gb[4];   // bins; a sample that is not valid lies above all of them
#pragma unroll
        for (int c = 0; c < 4; ++c) gb[c] = ok[c] ? (gk[c] - mn) >> sh : (uint32_t)kGuessBins;
        const int target = max(1, (kSpecQuantile * cnt + kGuessMaxK - 1) / kGuessMaxK);
        uint32_t bin = 0;   // the largest bin with fewer than `target` samples below it
#pragma unroll
        for (uint32_t bit = kGuessBins / 2; bit; bit >>= 1) {
            const uint32_t t = bin | bit;
            const int below = (int)(__popcll(__ballot(gb[0] < t)) + __popcll(__ballot(gb[1] < t)) +
                                    __popcll(__ballot(gb[2] < t)) + __popcll(__ballot(gb[3] < t)));
            bin = below < target ? t : bin;
        }
        ts = mn + (bin << sh);
    }
    return GuessStats{ts, cnt, mn, mx, sum};
}

}  // namespace gvr_dev

#endif  // GVR_GUESS_H
