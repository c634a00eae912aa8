// The partitioning step (Alg. 1) of one chain by one wave; used by ppo_partition.hip and ppo_kpath.hip.
#pragma once
#include "ppo_common.h"

namespace ppo {

struct PartitionShared {
    double P[PPO_MAX_L + 1];                 // prefix sums of the weights
    unsigned char next[PPO_MAX_L + 1];       // end of the first segment of the best partition from layer i on
    unsigned char cut[PPO_MAX_L];            // the cuts
};

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ unsigned long long readlane_u64(unsigned long long v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}

// f[i] = min over e in (i, hi[i]] of (value(e), segments(e) + 1, e) with value(e) = (e < L ? t[e-1] : 0) + f[e], which
// does not depend on i: a sliding-window minimum whose window moves towards the chain's start.  Lane x holds the
// candidate ends x + 1 and x + 65.  An end that is not better than one entered later (a smaller one) never is again, so
// the ends still alive get strictly better with growing e and the best of a window is the last one in it: a comparison
// in every lane and a bit search per layer in place of a reduction over the lanes (ppo_min_sum_partition, per call: 50 x 50
// layers 47 -> 19 us, 4096 x 128 layers 163 -> 74 us).
// Returns the number of segments (0: no partition); sum, and S.cut[0 .. segments - 2].
__device__ inline int min_sum_partition_wave(const float* __restrict__ t, const float* __restrict__ m, int L, double cap,
                                             int lane, PartitionShared& S, double& sum) {
    const double inf = __longlong_as_double(0x7FF0000000000000ll);
    const float t0 = lane < L ? t[lane] : 0.0f, t1 = lane + 64 < L ? t[lane + 64] : 0.0f;
    const float m0 = lane < L ? m[lane] : 0.0f, m1 = lane + 64 < L ? m[lane + 64] : 0.0f;
    auto at = [](float v0, float v1, int i) -> float {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(i < 64 ? v0 : v1), i & 63));
    };
    double acc = 0.0;
    S.P[0] = 0.0;
    for (int i = 0; i < L; ++i) {
        acc = acc + (double)at(m0, m1, i);
        S.P[i + 1] = acc;
    }
    wave_lds_fence();
    int top[2];   // last end that fits a segment starting at layer lane, lane + 64 (the layer itself if none)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = lane + 64 * h < L ? lane + 64 * h : L - 1;
        int lo = i, hi = L;
        while (lo < hi) {
            const int e = (lo + hi + 1) >> 1;
            if ((S.P[e] - S.P[i]) <= cap) lo = e; else hi = e - 1;
        }
        top[h] = lo;
    }
    double s0 = inf, s1 = inf;
    uint32_t k0 = 0, k1 = 0;                   // segments << 8 | end
    unsigned long long alive0 = 0, alive1 = 0;
    double f = 0.0;
    uint32_t segs = 0;
    for (int i = L - 1; i >= 0; --i) {
        if (f != inf) {                        // the end i + 1 enters
            const double s = (i + 1 < L ? (double)at(t0, t1, i) : 0.0) + f;
            const uint32_t key = ((segs + 1u) << 8) | (uint32_t)(i + 1);
            alive0 &= __ballot(s0 < s || (s0 == s && k0 < key));
            alive1 &= __ballot(s1 < s || (s1 == s && k1 < key));
            if (i < 64) {
                alive0 |= 1ull << i;
                if (lane == i) { s0 = s; k0 = key; }
            } else {
                alive1 |= 1ull << (i - 64);
                if (lane == i - 64) { s1 = s; k1 = key; }
            }
        }
        const int end = __builtin_amdgcn_readlane(i < 64 ? top[0] : top[1], i & 63);
        // ends up to `end` are the bits up to end - 1
        const unsigned long long in0 = end >= 64 ? alive0 : alive0 & ((1ull << end) - 1ull);
        const unsigned long long in1 = end <= 64 ? 0ull : end >= 128 ? alive1 : alive1 & ((1ull << (end - 64)) - 1ull);
        uint32_t key = (uint32_t)L;
        f = inf;
        if (in1) {
            const int x = 63 - __clzll((long long)in1);
            f = __longlong_as_double((long long)readlane_u64((unsigned long long)__double_as_longlong(s1), x));
            key = (uint32_t)__builtin_amdgcn_readlane((int)k1, x);
        } else if (in0) {
            const int x = 63 - __clzll((long long)in0);
            f = __longlong_as_double((long long)readlane_u64((unsigned long long)__double_as_longlong(s0), x));
            key = (uint32_t)__builtin_amdgcn_readlane((int)k0, x);
        }
        if (f == inf) key = (uint32_t)L;
        segs = key >> 8;
        S.next[i] = (unsigned char)(key & 0xFFu);
    }
    wave_lds_fence();
    sum = f;
    if (f == inf) return 0;
    int c = 0;
    for (int e = S.next[0]; e < L; e = S.next[e]) S.cut[c++] = (unsigned char)e;
    wave_lds_fence();
    return (int)segs;
}

}  // namespace ppo
