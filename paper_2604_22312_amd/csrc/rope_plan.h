// rope_plan.h -- planning of the static prior's kernels and the select's
// linear bins. Plain C++ with no HIP dependency, so the library and a
// sanitizer build on the CPU compile the same code.
#ifndef GVR_ROPE_PLAN_H
#define GVR_ROPE_PLAN_H

#include <stdint.h>

namespace gvr_rope {

constexpr int64_t kMaxN = ((int64_t)1 << 31) - 16;   // longest g (the header's GVR_ERR_TOO_LONG bound)

// The g kernel: kGPer positions per workgroup, one or kGLanes lanes for each.
constexpr int kGPer = 256;
constexpr int kGLanes = 4;

struct GLaunch {
    int lanes;        // lanes per position
    int64_t blocks;   // workgroups of kGPer * lanes threads
};

// Four lanes per position while all their waves are resident at once (131072
// positions are eight waves on each of 1024 SIMDs), and for longer where a
// position has many pairs; one from there on, and below four pairs, where
// lanes would idle. Measured (four lanes / one, us): d = 64, 131072 positions
// 12.7 / 13.9, 196608 18.1 / 17.4, 1048576 81.0 / 65.9; d = 512, 262144
// 128.1 / 137.1, 800000 398.3 / 391.3; d = 2, 1048576 28.8 / 11.1. A launch's
// threads must fit 32 bits, which four lanes per position of kMaxN would not.
inline GLaunch plan_g(int64_t n, int pairs) {
    const int64_t most = ((int64_t)1 << 17) * (pairs >= 128 ? pairs / 64 : 1);
    return GLaunch{n <= most && pairs >= kGLanes ? kGLanes : 1, n > 0 ? (n + kGPer - 1) / kGPer : 1};
}

// v's bin among kLinBins linear ones over [-lim, lim], with half = kLinBins / 2
// and scale = half / lim: non-decreasing in v (the fused multiply-add rounds
// monotonically), anything outside clamped, NaN in bin 0. Clamped before the
// conversion, which is undefined outside int's range. In float32, because the
// float64 form took much of both passes (prior at 131072 positions 57.2 ->
// 53.9 us).
constexpr int kLinBins = 2048;
constexpr int kInBin = 1024;   // most elements of the K-th one's bin
inline int lin_bin(float v, float half, float scale) {
    return (int)__builtin_fminf(__builtin_fmaxf(__builtin_fmaf(v, scale, half), 0.f), (float)(kLinBins - 1));
}

// Whether the binned select can serve a call: a wave's share must count in 16
// bits, and the K-th one's bin must hold at most kInBin elements, or a whole
// pass over g is spent before the radix select runs. That fails for finite g
// with one rotary pair (d = 2): g = 2 cos is crowded at its ends, its top bin
// holds acos(1 - 2 / (kLinBins / 2)) / pi = 1 / 71 of the positions, and once
// that is more than kInBin the bin below, 1 / 172 of them, is too, unless it
// lies above K. (K = 2048, radix / binned and then radix, us: 400000
// positions 516 / 565, 900000 1846 / 1953; the binned select alone at 131072:
// 107 against 175.) With more pairs the ends are thin.
constexpr int kSelectWaves = 16;
constexpr int64_t kMaxBinned = (int64_t)kSelectWaves * 61440;
inline bool binned_serves(int64_t n, int K, int pairs) {
    if (n > kMaxBinned) return false;
    const int64_t top = n / 71;   // of one pair
    return pairs > 1 || top <= kInBin || top < K;
}

}  // namespace gvr_rope

#endif  // GVR_ROPE_PLAN_H
