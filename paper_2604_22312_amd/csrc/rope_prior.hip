// rope_prior.hip -- the static RoPE/YaRN prior P_static (Sec. 3.2, 3.3) on
// MI355X (gfx950), behind the C ABI declared in include/gvr_rope_prior.h.
//
//   g kernel. One or four lanes per relative position Delta (workgroups of
//   256 positions; rope_plan.h says which). The first d/2 threads of every
//   workgroup derive the YaRN angles theta'_i into LDS (a few pow/log calls,
//   the same in every workgroup), then the lanes of a position sum
//   cos(Delta * theta'_i) in float64, as four sums of every fourth pair added
//   as (0 + 1) + (2 + 3). Bound by the latency of the float64 cosines until
//   the positions alone fill the compute units (d = 64: 131072 positions 12.7
//   us with four lanes each, 13.9 with one), by their rate from there on
//   (1048576 positions 65.9 us with one lane each, 81.0 with four). Run once
//   per model and length, not per decode step.
//
//   select kernel. One workgroup of 1024 threads: the calls take no scratch
//   memory that several could meet in (only out_delta's K words are unused
//   until the select writes them). So it is bound by one compute unit's read
//   rate and reads g twice. The first pass counts every element
//   into linear bins over [-d, d] (g cannot leave it), one histogram per wave:
//   that gives the bin holding the K-th largest g and the place of each
//   wave's elements at or above it. The second lists the indices of those, in
//   index order, and the keys of the bin's own elements, which are ranked
//   among themselves (lower index first); a block scan writes the selected
//   indices. (A radix select over the 64-bit keys read g four or five times
//   with one load in flight: the prior of 131072 positions took 220 us, now
//   46, of which the g kernel takes 14.) It remains for what the bins cannot
//   serve (binned_serves of rope_plan.h says what is known ahead; the rest,
//   NaN among it, is found by the first pass). Digits of 11, 11, 11, 11, 10,
//   10 bits of the order-preserving key; as soon as the elements sharing the selected prefix
//   fit in LDS (<= 4096) they are gathered there; a final pass in index order
//   writes the selection at offsets from two block scans per 4096 elements.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "gvr_rope_prior.h"
#pragma clang force_cuda_host_device begin
#include "rope_plan.h"
#pragma clang force_cuda_host_device end

#define DEV __device__ __forceinline__

namespace {

using gvr_rope::kGLanes;
using gvr_rope::kGPer;
using gvr_rope::kInBin;
using gvr_rope::kLinBins;
using gvr_rope::kMaxN;
using gvr_rope::lin_bin;

constexpr int kMaxPairs = 256;               // d <= 512
constexpr int kSBlock = 1024;                // threads of the select workgroup
constexpr int kSWaves = kSBlock / 64;
constexpr int kSelBins = 2048;               // widest digit: 11 bits
constexpr int kGather = 4096;                // keys the select keeps in LDS
constexpr int kDigits = 6;
constexpr int kEmitPer = 4;                  // consecutive elements per thread in the emit pass

__constant__ int kDigitShift[kDigits] = {53, 42, 31, 20, 10, 0};
__constant__ int kDigitBits[kDigits] = {11, 11, 11, 11, 10, 10};

struct RopeArgs {
    int d;
    int orig_ctx;
    double base, scale, beta_fast, beta_slow;
};

// theta'_i of one rotary pair (YaRN ramp over the pair index).
DEV double yarn_angle(int i, const RopeArgs& a) {
#pragma clang fp contract(off)
    const double two_pi = 6.283185307179586;
    const double ln_base = log(a.base);
    const double x_fast = a.d * log(a.orig_ctx / (two_pi * a.beta_fast)) / (2.0 * ln_base);
    const double x_slow = a.d * log(a.orig_ctx / (two_pi * a.beta_slow)) / (2.0 * ln_base);
    const double lo = fmax(floor(x_fast), 0.0);
    const double hi = fmin(ceil(x_slow), (double)(a.d - 1));
    const double theta = pow(a.base, -2.0 * i / a.d);
    const double gamma = fmin(fmax((i - lo) / fmax(hi - lo, 1e-3), 0.0), 1.0);
    return theta * (1.0 - gamma) + (theta / a.scale) * gamma;
}

template <int LANES>
__global__ __launch_bounds__(kGPer * LANES) void rope_g_kernel(int64_t n, RopeArgs a, double* __restrict__ g,
                                                               double* __restrict__ theta_out) {
    __shared__ double th[kMaxPairs];
    const int h = a.d / 2;
    const int t = threadIdx.x;
    if (t < h) {
        const double v = yarn_angle(t, a);
        th[t] = v;
        if (blockIdx.x == 0 && theta_out) theta_out[t] = v;
    }
    __syncthreads();
    const int64_t delta = (int64_t)blockIdx.x * kGPer + t / LANES;
    const double x = (double)delta;
    // Four sums, of every fourth pair each, added as (0 + 1) + (2 + 3) in both
    // forms: g(Delta) is the same bits for every n.
    auto every_fourth = [&](int q) {
        double acc = 0.0;
        for (int i = q; i < h; i += kGLanes) acc += cos(x * th[i]);
        return acc;
    };
    double acc = 0.0;
    if constexpr (LANES == kGLanes) {
        acc = every_fourth(t % kGLanes);
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
    } else {
#pragma unroll 1
        for (int q = 0; q < kGLanes && q < h; q += 2) {
            const double even = every_fourth(q);
            acc += even + every_fourth(q + 1);
        }
    }
    if (delta < n && t % LANES == 0) g[delta] = 2.0 * acc;
}

// Order-preserving 64-bit key of a float64 (-0.0 folded into +0.0 first).
DEV uint64_t order_key(double v) {
    v = v + 0.0;
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Exclusive prefix sum of v over the workgroup's threads in thread order;
// *total receives the sum over all threads. Every thread must call it.
DEV uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum, uint32_t* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t base = 0, tot = 0;
    for (int i = 0; i < kSWaves; ++i) {
        const uint32_t s = wsum[i];
        base += (i < w) ? s : 0u;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + x - v;
}

// The binned select (see the file comment). Returns false, with nothing
// written, where it does not apply; every thread returns the same.
constexpr int kList = GVR_MAX_K + kInBin;    // listed: fewer than K above the K-th one's bin, and the bin
constexpr int kPairs = 8;                    // 16-byte loads in flight per lane
static_assert(kSWaves == gvr_rope::kSelectWaves, "a wave's share counts in 16 bits");
struct BinnedSmem {
    uint32_t hist[kSWaves][kLinBins / 2];    // two 16-bit counts per word
    uint32_t list[kList];                    // index, bit 31: in the K-th one's bin and not (yet) selected
    uint64_t key[kInBin];
    uint32_t pos[kInBin];                    // place in the list
    uint32_t wcnt[kSWaves];
    uint32_t wsum[kSWaves];
    uint32_t bin, above, cnt, fill, bad;
};
typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));

// One wave's elements [w0, w1) of g in pairs, kPairs 128-element chunks in
// flight; body(v, i, full) gets elements i and i + 1, all inside the range if
// `full` (a compile-time constant), else masked by i < w1 and i + 1 < w1.
template <typename Body>
DEV void stream_pairs(const double* __restrict__ g, int n, int w0, int w1, int lane, Body&& body) {
    int b = w0;
    for (; b + 128 * kPairs <= w1; b += 128 * kPairs) {
        const double* gb = g + b + 2 * lane;
        d2 v[kPairs];
#pragma unroll
        for (int u = 0; u < kPairs; ++u) v[u] = *reinterpret_cast<const d2*>(gb + 128 * u);
#pragma unroll
        for (int u = 0; u < kPairs; ++u) body(v[u], b + 128 * u + 2 * lane, std::true_type{});
    }
    for (; b < w1; b += 128) {
        const int i = b + 2 * lane;
        d2 v = *reinterpret_cast<const d2*>(g + min(i, n - 2));   // (n >= 2) the last pair again past the end
        if (i == n - 1) v.x = v.y;
        body(v, i, std::false_type{});
    }
}

DEV bool binned_select(BinnedSmem& sm, const double* __restrict__ g, int n, int K, float lim,
                       int32_t* __restrict__ out) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float half = 0.5f * kLinBins, scale = half / lim;
    const int share = ((n + kSWaves - 1) / kSWaves + 127) / 128 * 128;
    const int w0 = min(wave * share, n), w1 = min(w0 + share, n);
    for (int i = tid; i < kSWaves * kLinBins / 2; i += kSBlock) (&sm.hist[0][0])[i] = 0;
    if (tid == 0) {
        sm.bad = 0;
        sm.fill = 0;
    }
    __syncthreads();
    // Pass 1: count every element.
    uint32_t* const hw = sm.hist[wave];
    bool bad = false;
    stream_pairs(g, n, w0, w1, lane, [&](const d2& v, int i, auto full) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float e = (float)(c ? v.y : v.x);
            if (full.value || i + c < w1) {
                bad |= e != e;   // NaN: ordered by its sign, not by a bin
                const int b = lin_bin(e, half, scale);
                atomicAdd(&hw[b >> 1], 1u << (16 * (b & 1)));
            }
        }
    });
    if (bad) sm.bad = 1;
    __syncthreads();
    if (sm.bad) return false;
    // Thread t holds bins kLinBins - 1 - 2t and the one below: a scan in
    // thread order counts the elements in higher bins.
    const int word = kLinBins / 2 - 1 - tid;   // kSBlock words
    static_assert(kLinBins / 2 == kSBlock, "one histogram word per thread");
    uint32_t lo = 0, hi = 0;
    for (int w = 0; w < kSWaves; ++w) {
        const uint32_t c = sm.hist[w][word];
        lo += c & 0xFFFFu;
        hi += c >> 16;
    }
    uint32_t tot;
    const uint32_t above = block_exclusive_scan(lo + hi, sm.wsum, &tot);
    const uint32_t k = (uint32_t)K;
    if (above < k && k <= above + lo + hi) {
        const bool up = k <= above + hi;
        sm.bin = (uint32_t)(2 * word + (up ? 1 : 0));
        sm.above = up ? above : above + hi;
        sm.cnt = up ? hi : lo;
    }
    __syncthreads();
    const int bin = (int)sm.bin;
    const uint32_t nab = sm.above, nin = sm.cnt;
    if (nin > (uint32_t)kInBin) return false;   // (nab < K)
    // Each wave's elements at or above the bin (pairs of bins; the bin's word
    // counts both of its bins only if it is the lower one).
    uint32_t mine = 0;
    for (int j = bin / 2 + lane; j < kLinBins / 2; j += 64) {
        const uint32_t c = hw[j];
        mine += (c >> 16) + (2 * j >= bin ? c & 0xFFFFu : 0u);
    }
    for (int o = 32; o; o >>= 1) mine += __shfl_xor(mine, o, 64);
    if (lane == 0) sm.wcnt[wave] = mine;
    __syncthreads();
    uint32_t at = 0;
    for (int w = 0; w < wave; ++w) at += sm.wcnt[w];
    // Pass 2: list them in index order.
    const uint64_t below = lane ? ~0ull >> (64 - lane) : 0ull;   // lanes below this one
    stream_pairs(g, n, w0, w1, lane, [&](const d2& v, int i, auto full) {
        const int b0 = full.value || i < w1 ? lin_bin((float)v.x, half, scale) : -1;
        const int b1 = full.value || i + 1 < w1 ? lin_bin((float)v.y, half, scale) : -1;
        const uint64_t m0 = __ballot(b0 >= bin), m1 = __ballot(b1 >= bin);
        if (m0 | m1) {   // (wave-uniform)
            uint32_t p = at + (uint32_t)(__popcll(m0 & below) + __popcll(m1 & below));
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int b = c ? b1 : b0;
                if (b >= bin) {
                    sm.list[p] = (uint32_t)(i + c) | (b == bin ? 0x80000000u : 0u);
                    if (b == bin) {
                        const uint32_t q = atomicAdd(&sm.fill, 1u);
                        sm.key[q] = order_key(c ? v.y : v.x);
                        sm.pos[q] = p;
                    }
                    ++p;
                }
            }
            at += (uint32_t)(__popcll(m0) + __popcll(m1));
        }
    });
    __syncthreads();
    // The bin's elements: the K - nab largest, the lower index first among equals.
    if (tid < (int)nin) {
        const uint64_t kk = sm.key[tid];
        const uint32_t pp = sm.pos[tid];
        uint32_t before = 0;
        for (uint32_t j = 0; j < nin; ++j) {
            const uint64_t o = sm.key[j];
            before += o > kk || (o == kk && sm.pos[j] < pp);
        }
        if (before < k - nab) sm.list[pp] &= 0x7FFFFFFFu;
    }
    __syncthreads();
    static_assert(kList % kSBlock == 0, "whole list entries per thread");
    constexpr int kPer = kList / kSBlock;
    const uint32_t m = nab + nin;
    uint32_t e[kPer], take = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t q = (uint32_t)(tid * kPer + j);
        e[j] = q < m ? sm.list[q] : 0x80000000u;
        take += !(e[j] >> 31);
    }
    uint32_t p = block_exclusive_scan(take, sm.wsum, &tot);
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (!(e[j] >> 31)) out[p++] = (int32_t)e[j];
    return true;
}

// BINNED: the binned select, and the radix select where it gives up; else the
// radix select alone.
template <bool BINNED>
__global__ __launch_bounds__(kSBlock) void prior_select_kernel(const double* __restrict__ g, int64_t n, int K,
                                                               float lim, int32_t* __restrict__ out) {
    struct RadixSmem {
        uint32_t hist[kSelBins];
        uint64_t cand[kGather];
        uint32_t wsum[kSWaves];
        uint32_t bin, need, cnt, ncand;
    };
    union BothSmem {
        BinnedSmem b;
        RadixSmem r;
    };
    __shared__ std::conditional_t<BINNED, BothSmem, RadixSmem> sm;
    RadixSmem& r = [&]() -> RadixSmem& {
        if constexpr (BINNED) return sm.r;
        else return sm;
    }();
    uint32_t* const hist = r.hist;
    uint64_t* const cand = r.cand;
    uint32_t* const wsum = r.wsum;
    uint32_t &s_bin = r.bin, &s_need = r.need, &s_cnt = r.cnt, &s_ncand = r.ncand;
    const int tid = threadIdx.x;
    if (n <= K) {
        for (int i = tid; i < K; i += kSBlock) out[i] = (i < n) ? i : -1;
        return;
    }
    if constexpr (BINNED) {
        if (binned_select(sm.b, g, (int)n, K, lim, out)) return;
        __syncthreads();   // the binned select's arrays are dead
    }
    uint64_t prefix = 0, mask = 0;
    uint32_t need = (uint32_t)K;     // rank of the K-th key among those sharing `prefix`
    uint32_t ncand = 0;
    bool in_lds = false;
    for (int dg = 0; dg < kDigits; ++dg) {
        const int sh = kDigitShift[dg];
        const int nb = 1 << kDigitBits[dg];
        for (int b = tid; b < nb; b += kSBlock) hist[b] = 0;
        __syncthreads();
        if (in_lds) {
            for (uint32_t i = tid; i < ncand; i += kSBlock) {
                const uint64_t k = cand[i];
                if ((k & mask) == prefix) atomicAdd(&hist[(k >> sh) & (uint64_t)(nb - 1)], 1u);
            }
        } else {
            for (int64_t i = tid; i < n; i += kSBlock) {
                const uint64_t k = order_key(g[i]);
                if ((k & mask) == prefix) atomicAdd(&hist[(k >> sh) & (uint64_t)(nb - 1)], 1u);
            }
        }
        __syncthreads();
        // Thread t holds bins nb-1-2t and nb-2-2t (descending), so a scan in
        // thread order counts the keys in higher bins.
        const int b0 = nb - 1 - 2 * tid, b1 = b0 - 1;
        const uint32_t c0 = (b0 >= 0) ? hist[b0] : 0u;
        const uint32_t c1 = (b1 >= 0) ? hist[b1] : 0u;
        uint32_t tot;
        const uint32_t above = block_exclusive_scan(c0 + c1, wsum, &tot);
        if (above < need && need <= above + c0 + c1) {
            if (need <= above + c0) {
                s_bin = (uint32_t)b0; s_need = need - above; s_cnt = c0;
            } else {
                s_bin = (uint32_t)b1; s_need = need - above - c0; s_cnt = c1;
            }
        }
        __syncthreads();
        prefix |= (uint64_t)s_bin << sh;
        mask |= (uint64_t)(nb - 1) << sh;
        need = s_need;
        const uint32_t cnt = s_cnt;
        __syncthreads();
        if (!in_lds && cnt <= (uint32_t)kGather && dg + 1 < kDigits) {
            if (tid == 0) s_ncand = 0;
            __syncthreads();
            for (int64_t i = tid; i < n; i += kSBlock) {
                const uint64_t k = order_key(g[i]);
                if ((k & mask) == prefix) {
                    const uint32_t slot = atomicAdd(&s_ncand, 1u);
                    if (slot < (uint32_t)kGather) cand[slot] = k;
                }
            }
            __syncthreads();
            ncand = s_ncand;
            in_lds = true;
        }
    }
    // prefix is now the K-th largest key; `need` keys equal to it are taken,
    // the lowest indices first.
    const uint64_t kth = prefix;
    uint32_t carry_eq = 0, carry_sel = 0;
    for (int64_t base = 0; base < n; base += (int64_t)kSBlock * kEmitPer) {
        const int64_t i0 = base + (int64_t)tid * kEmitPer;
        uint32_t gt = 0, eq = 0;   // bit j: element i0 + j beats / equals the K-th key
        for (int j = 0; j < kEmitPer; ++j) {
            if (i0 + j < n) {
                const uint64_t k = order_key(g[i0 + j]);
                gt |= (uint32_t)(k > kth) << j;
                eq |= (uint32_t)(k == kth) << j;
            }
        }
        uint32_t tot_eq;
        uint32_t rank = carry_eq + block_exclusive_scan((uint32_t)__builtin_popcount(eq), wsum, &tot_eq);
        uint32_t sel = gt;
        for (int j = 0; j < kEmitPer; ++j) {
            if ((eq >> j) & 1u) {
                if (rank < need) sel |= 1u << j;
                ++rank;
            }
        }
        uint32_t tot_sel;
        uint32_t pos = carry_sel + block_exclusive_scan((uint32_t)__builtin_popcount(sel), wsum, &tot_sel);
        for (int j = 0; j < kEmitPer; ++j) {
            if (((sel >> j) & 1u) && pos < (uint32_t)K) out[pos++] = (int32_t)(i0 + j);
        }
        carry_eq += tot_eq;
        carry_sel += tot_sel;
    }
}

bool finite_pos(double v) { return isfinite(v) && v > 0.0; }

gvr_status read_params(const gvr_rope_params* p, RopeArgs* a) {
    gvr_rope_params d;
    if (!p) {
        gvr_rope_params_default(&d);
        p = &d;
    }
    if (p->d_rope < 2 || p->d_rope > 2 * kMaxPairs || (p->d_rope & 1)) return GVR_ERR_INVALID_ARG;
    if (p->orig_ctx < 1) return GVR_ERR_INVALID_ARG;
    if (!isfinite(p->base) || p->base <= 1.0) return GVR_ERR_INVALID_ARG;
    if (!finite_pos(p->scale) || !finite_pos(p->beta_fast) || !finite_pos(p->beta_slow)) return GVR_ERR_INVALID_ARG;
    a->d = p->d_rope;
    a->orig_ctx = p->orig_ctx;
    a->base = p->base;
    a->scale = p->scale;
    a->beta_fast = p->beta_fast;
    a->beta_slow = p->beta_slow;
    return GVR_OK;
}

gvr_status launch_g(int64_t n, const RopeArgs& a, double* g, double* theta, void* stream) {
    const gvr_rope::GLaunch p = gvr_rope::plan_g(n, a.d / 2);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)p.blocks), dim3((unsigned)(kGPer * p.lanes)), 0, (hipStream_t)stream,
                           n, a, g, theta);
    };
    p.lanes == kGLanes ? launch(rope_g_kernel<kGLanes>) : launch(rope_g_kernel<1>);
    return hipGetLastError() == hipSuccess ? GVR_OK : GVR_ERR_HIP;
}

}  // namespace

extern "C" {

void gvr_rope_params_default(gvr_rope_params* p) {
    if (!p) return;
    p->d_rope = 64;
    p->orig_ctx = 4096;
    p->base = 10000.0;
    p->scale = 40.0;
    p->beta_fast = 32.0;
    p->beta_slow = 1.0;
}

gvr_status gvr_rope_g(int64_t n, const gvr_rope_params* params, double* g, double* theta, void* stream) {
    RopeArgs a;
    const gvr_status st = read_params(params, &a);
    if (st != GVR_OK) return st;
    if (n < 0 || (n > 0 && !g)) return GVR_ERR_INVALID_ARG;
    if (n > kMaxN) return GVR_ERR_TOO_LONG;
    if (n == 0 && !theta) return GVR_OK;
    return launch_g(n, a, g, theta, stream);
}

gvr_status gvr_rope_prior(int64_t n, int32_t K, const gvr_rope_params* params, double* g, int32_t* out_delta,
                          void* stream) {
    RopeArgs a;
    const gvr_status st = read_params(params, &a);
    if (st != GVR_OK) return st;
    if (n < 0 || (n > 0 && !g) || !out_delta) return GVR_ERR_INVALID_ARG;
    if (K < 1 || K > GVR_MAX_K) return GVR_ERR_UNSUPPORTED_K;
    if (n > kMaxN) return GVR_ERR_TOO_LONG;
    if (n > 0) {
        const gvr_status s = launch_g(n, a, g, nullptr, stream);
        if (s != GVR_OK) return s;
    }
    const bool binned = gvr_rope::binned_serves(n, K, a.d / 2);
    hipLaunchKernelGGL(binned ? prior_select_kernel<true> : prior_select_kernel<false>, dim3(1), dim3(kSBlock), 0,
                       (hipStream_t)stream, (const double*)g, n, (int)K, (float)a.d, out_delta);
    return hipGetLastError() == hipSuccess ? GVR_OK : GVR_ERR_HIP;
}

}  // extern "C"
