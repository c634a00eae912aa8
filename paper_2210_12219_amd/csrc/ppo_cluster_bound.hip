// Cluster form: what a search can leave out.  Most nodes and cuts of a cluster cannot be part of an optimum: nearly all
// links are slower than the bottleneck of a good placement.  Two kernels before the levels of ppo_cluster.hip find that out.
//
// cluster_bound_kernel: a placement on nine nodes of the cluster.  Any placement's bottleneck is an upper bound U of the
// optimum; the best one on nine well connected nodes, cutting at the 31 smallest transfer sizes, is the optimum itself or a
// few per cent above it (20 nodes of mixed capacities: equal in one of three instances, 1.21 times at most).
// Two choices of nodes, a workgroup each: by the three fastest links, and by links and capacity together.
//
// cluster_reduce_kernel: only cuts and links with a quotient of at most U can matter.  Over those, dropping the rule that a
// node is used once leaves walks: back[j] = cuts from which a walk that starts a segment on j there reaches the end,
// fore[j] = cuts at which a walk from the start of the chain starts a segment on j.  Every placement with a bottleneck of at
// most U is such a walk, so a node j with fore[j] & back[j] empty, and a cut in none of them, is in none of these; all
// optima and their ties are kept.  The search then runs on the nodes and cuts that are left, in their order: 20 nodes and
// 100 layers become 9 to 16 nodes and 10 to 18 layers, 10.5 million rows of 100 entries 2 to 520 thousand of 10 to 18.  An
// instance without a placement on the nine nodes, or with more than 62 cuts left, is searched whole.
//
// The search for few segments (ppo_cluster_few.hip) goes the same way, with up to 64 nodes, segments counted, and the bound
// itself handed on.
//
// What bounds these two: the one workgroup's instruction issue in the levels of the first (2304 rows, 22 of its 30 us) and
// chains of LDS reads and barriers in the second (24 to 28 us).  One cluster of 20 nodes and 100 layers: 2040 us a call without
// them, 120 to 320 with them, by how much can be left out; 32 of 15 devices and 50 layers: 827 and 480 to 500 (no node and two
// thirds of the layers left out).  What they cost where nothing can be: beside cluster_confined and few_confined.
#include "ppo_cluster.h"
#include "ppo_sets.h"

namespace ppo {

namespace {

typedef unsigned short b_us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t b_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(b_us2, a), __builtin_bit_cast(b_us2, b)));
}
__device__ __forceinline__ uint32_t b_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(b_us2, a), __builtin_bit_cast(b_us2, b)));
}

constexpr int kBoundNodes = 9, kBoundThreads = 1024, kBoundWaves = kBoundThreads / 64;
constexpr int kBoundEntries = 32, kBoundRow = kBoundEntries / 2;   // the start of the chain and 31 cuts; dwords of a row
constexpr uint32_t kBoundInf = kInfBits >> 16;                     // codes: the upper half of the pattern, rounded up
constexpr int kMostCuts = 62;                                      // that the walks take: a bit each, and the chain's start
constexpr int kBoundRuns = 5;                                      // minima over runs of 1 .. 16 entries
constexpr int kBoundPad = 52;                                      // dwords of +inf, then of 0, after the runs of a wave
constexpr int kBoundRunDwords = kBoundRuns * 64 + 2 * kBoundPad;
constexpr uint32_t kBoundNone = kBoundRuns * 256u, kBoundEnds = kBoundNone + kBoundPad * 4u;   // byte offsets of those
__host__ __device__ constexpr int bound_level_rows(int c) { return (int)kSetsHost.choose[kBoundNodes][c] * c; }
constexpr int kBoundOddRows = 630, kBoundEvenRows = 504;           // the widest levels of odd and of even size
static_assert(bound_level_rows(5) == kBoundOddRows && bound_level_rows(3) <= kBoundOddRows && bound_level_rows(7) <= kBoundOddRows &&
              bound_level_rows(4) == kBoundEvenRows && bound_level_rows(6) <= kBoundEvenRows && bound_level_rows(2) <= kBoundEvenRows &&
              bound_level_rows(8) <= kBoundEvenRows && bound_level_rows(9) <= kBoundOddRows, "rows of two levels at a time");

struct BoundShared {
    double P[PPO_MAX_L + 64 + 1];                  // written 64 at a time
    float t[PPO_MAX_L], m[PPO_MAX_L], M[PPO_CLUSTER_FEW_MAX_N], B[PPO_CLUSTER_FEW_MAX_N * PPO_CLUSTER_FEW_MAX_N];
    unsigned long long cuts[2];                    // bit e: the cut e is one of the 31
    uint32_t best;
    int least[2];                                  // cuts with the least transfer size of all
    int level[kBoundNodes + 2];
    unsigned char node[16], pos[kBoundEntries];    // cluster nodes and cuts of the small search; pos[0] = 0
    uint16_t order[1 << kBoundNodes], place[1 << kBoundNodes];
    uint32_t query[kBoundNodes][kBoundEntries];    // windows: byte offsets of two runs that cover them, 16 bits each
    uint16_t q[kBoundNodes][kBoundNodes][kBoundEntries];
    uint32_t run[kBoundWaves][kBoundRunDwords];
    uint32_t rows[(kBoundOddRows + kBoundEvenRows) * kBoundRow];
};
static_assert(sizeof(BoundShared) <= 160 * 1024, "one workgroup to a compute unit");

// Prefix sums in index order in binary64 by one wave: a lane's weight is fetched from its register.
__device__ __forceinline__ void prefix_sums(const float* m_s, int L, int lane, double* P) {
    double acc = 0.0;
    P[0] = 0.0;
    for (int base = 0; base < L; base += 64) {
        const float w = base + lane < L ? m_s[base + lane] : 0.0f;
        for (int from = 0; from < 64 && base + from < L; from += 16)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc = acc + (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), from + i));
                P[base + from + i + 1] = acc;
            }
    }
}

// the last end e' such that layers [e, e') fit (e if none): the ends that fit grow with e, so a binary search finds it
__device__ __forceinline__ int window_end(const double* P, int L, double cap, int e) {
    int good = e, step = 1;
    const double at = P[e];
    while (step < L) step <<= 1;
    for (; step >= 1; step >>= 1) {
        const int e2 = good + step;
        if (e2 <= L && P[e2] - at <= cap) good = e2;
    }
    return good;
}

// cuts 0 .. e of a set of cuts, counted
__device__ __forceinline__ int cuts_upto(unsigned long long c0, unsigned long long c1, int e) {
    const unsigned long long m0 = e >= 63 ? ~0ull : (2ull << e) - 1ull, m1 = e < 64 ? 0ull : e >= 127 ? ~0ull : (2ull << (e - 64)) - 1ull;
    return __popcll(c0 & m0) + __popcll(c1 & m1);
}

template <int C>
__device__ __forceinline__ void bound_level(BoundShared& s, int lane, int wave) {
    const int hl = lane & 15, part = lane >> 4;
    uint32_t* from = s.rows + (C & 1 ? 0 : kBoundOddRows * kBoundRow);
    uint32_t* to = s.rows + (C & 1 ? kBoundOddRows * kBoundRow : 0);
    constexpr int nsets = (int)kSetsHost.choose[kBoundNodes][C], groups = (nsets + 3) / 4;
    uint32_t* run32 = s.run[wave];
    const unsigned char* runb = reinterpret_cast<const unsigned char*>(run32) + part * 64;
    const uint32_t* q32 = reinterpret_cast<const uint32_t*>(s.q);
    // a wave takes one node outside of a group of four sets at a time
    for (int it = wave; it < groups * (kBoundNodes - C); it += kBoundWaves) {
        const int group = it % groups, skip = it / groups;
        const int idx = group * 4 + part;
        const bool mine = idx < nsets;
        const uint32_t mp = s.order[s.level[C] + (mine ? idx : nsets - 1)];
        uint32_t jb = ((1u << kBoundNodes) - 1u) & ~mp;
        for (int i = 0; i < skip; ++i) jb &= jb - 1u;
        const uint32_t j = (uint32_t)__builtin_ctz(jb), set = mp | (1u << j);
        const uint32_t first = (uint32_t)s.place[mp] * C;
        uint32_t v = kBoundInf | (kBoundInf << 16), bits = mp;
#pragma unroll
        for (int m = 0; m < C; ++m) {
            const uint32_t b = (uint32_t)__builtin_ctz(bits);
            bits &= bits - 1u;
            v = b_min(v, b_max(q32[(b * kBoundNodes + j) * kBoundRow + hl], from[(first + m) * kBoundRow + hl]));
        }
        // minima over runs of 2^r entries starting at each entry (shifts within the 16 lanes of a set)
        run32[lane] = v;
        const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x101, 0xF, 0xF, true);
        uint32_t cur = b_min(v, (v >> 16) | (next << 16));
        run32[64 + lane] = cur;
        cur = b_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x101, 0xF, 0xF, true));
        run32[128 + lane] = cur;
        cur = b_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x102, 0xF, 0xF, true));
        run32[192 + lane] = cur;
        cur = b_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x104, 0xF, 0xF, true));
        run32[256 + lane] = cur;
        const uint2 qd = *reinterpret_cast<const uint2*>(&s.query[j][2 * hl]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t res[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t d = h ? qd.y : qd.x;
            const uint32_t r1 = *reinterpret_cast<const uint16_t*>(runb + (d & 0xFFFFu));
            const uint32_t r2 = *reinterpret_cast<const uint16_t*>(runb + (d >> 16));
            res[h] = r1 < r2 ? r1 : r2;
        }
        const uint32_t row = (uint32_t)s.place[set] * (C + 1) + (uint32_t)__popc(mp & ((1u << j) - 1u));
        if (mine) to[row * kBoundRow + hl] = res[0] | (res[1] << 16);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
}

}  // namespace

static __constant__ SetValues kSetValues = SetValues();

__global__ __launch_bounds__(kBoundThreads) void cluster_bound_kernel(const float* __restrict__ t, const float* __restrict__ m,
                                                                     const float* __restrict__ M, const float* __restrict__ B,
                                                                     int L, int n, int pmax, unsigned char* __restrict__ out,
                                                                     size_t stride) {
    extern __shared__ __align__(16) unsigned char bound_sm[];
    BoundShared& s = *reinterpret_cast<BoundShared*>(bound_sm);
    const int inst = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < L) {
        const float x = t[(size_t)inst * L + tid];
        s.t[tid] = x == 0.0f ? 0.0f : x;   // -0 is a size of zero: +0
        s.m[tid] = m[(size_t)inst * L + tid];
    }
    if (tid < n) s.M[tid] = M[(size_t)inst * n + tid];
    if (tid == 0) s.best = kBoundInf;
    for (int i = tid; i < n * n; i += kBoundThreads) {
        const int a = i / n, b = i - a * n;   // the element with the smaller row index is the one read
        s.B[i] = B[(size_t)inst * n * n + (a < b ? i : b * n + a)];
    }
    uint32_t set_value = 0;
    if (tid < 1 << kBoundNodes) set_value = kSetValues.row_and_place[tid] >> 16;
    if (tid < kBoundNodes + 2) s.level[tid] = (int)kSetValues.level[kBoundNodes][tid];
    for (int i = lane; i < kBoundPad; i += 64) {
        s.run[wave][kBoundRuns * 64 + i] = kBoundInf | (kBoundInf << 16);
        s.run[wave][kBoundRuns * 64 + kBoundPad + i] = 0u;
    }
    __syncthreads();
    if (tid < 1 << kBoundNodes) {
        s.place[tid] = (uint16_t)set_value;
        s.order[s.level[__popc((uint32_t)tid)] + (int)set_value] = (uint16_t)tid;
    }
    if (wave == 0) {
        prefix_sums(s.m, L, lane, s.P);
    } else if (wave == 1) {
        // the nodes: by the mean of the three fastest links, or by four links and the capacity in logarithms
        float top[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int b = 0; b < n; ++b) {
            float x = lane < n && b != lane ? s.B[lane * n + b] : 0.0f;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float most = top[u] > x ? top[u] : x;
                x = top[u] > x ? x : top[u];
                top[u] = most;
            }
        }
        float score = top[0] + top[1] + top[2];
        if (blockIdx.x == 1)
            score = __log2f(top[0]) + __log2f(top[1]) + __log2f(top[2]) + __log2f(top[3]) + 2.0f * __log2f(lane < n ? s.M[lane] : 1.0f);
        int rank = 0;
        for (int b = 0; b < n; ++b) {
            const float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(score), b));
            rank += (x > score || (x == score && b < lane)) ? 1 : 0;
        }
        // (scores that are no numbers: the first nodes)
        unsigned long long chosen = __ballot(lane < n && rank < kBoundNodes);
        if (__popcll(chosen) != kBoundNodes) chosen = (1ull << kBoundNodes) - 1ull;
        if ((chosen >> lane) & 1ull) s.node[__popcll(chosen & ((1ull << lane) - 1ull))] = (unsigned char)lane;
    } else if (wave < 4) {
        // the cuts: after the layers with the smallest t (ties by index)
        const int i = (wave - 2) * 64 + lane;   // the cut i + 1
        int rank = 0, smaller = 0;
        const float x = i < L - 1 ? s.t[i] : 0.0f;
        for (int u = 0; u < L - 1; ++u) {
            smaller += s.t[u] < x ? 1 : 0;
            rank += (s.t[u] < x || (s.t[u] == x && u < i)) ? 1 : 0;
        }
        const unsigned long long some = __ballot(i < L - 1 && rank < kBoundEntries - 1), least = __ballot(i < L - 1 && smaller == 0);
        if (lane == 0) {
            s.cuts[wave - 2] = some;
            s.least[wave - 2] = __popcll(least);
        }
    }
    __syncthreads();
    // What cannot lead to a confined search ends here: nine nodes that do not hold the chain (as many of the largest as there
    // may be segments), or, where a link is needed, more cuts with the least transfer size than the walks take.  One cluster of 16
    // nodes and 100 layers whose nine best nodes are short of memory, in us: 252 without a bound, 293 with all of this, 271 so.
    {
        const int j = lane < kBoundNodes ? lane : 0, most = pmax < kBoundNodes ? pmax : kBoundNodes;
        const float cap = s.M[s.node[j]];
        int rank = 0;   // among the nine
        if (most < kBoundNodes)
#pragma unroll
            for (int b = 0; b < kBoundNodes; ++b) {
                const float other = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cap), b));
                rank += (other > cap || (other == cap && b < j)) ? 1 : 0;
            }
        double held = lane < kBoundNodes && rank < most ? (double)cap : 0.0;
        for (int off = 8; off >= 1; off >>= 1) held += __shfl_xor(held, off, 64);
        const bool alone = __ballot(lane < n && (double)s.M[lane < n ? lane : 0] >= s.P[L]) != 0ull;
        // (lanes 0 .. 15 have the sum; what is in doubt by a rounding is gone through)
        if (__ballot(lane == 0 && held < s.P[L]) != 0ull || (!alone && s.least[0] + s.least[1] > kMostCuts)) {
            if (tid == 0) reinterpret_cast<uint32_t*>(out + (size_t)inst * stride)[blockIdx.x] = kInfBits;
            return;
        }
    }
    // the cuts as bits (bit e), and in increasing order
    const unsigned long long c0 = s.cuts[0] << 1, c1 = s.cuts[1] << 1 | s.cuts[0] >> 63;
    const int count = __popcll(c0) + __popcll(c1);
    if (tid < 128 && tid >= 1 && ((tid < 64 ? c0 >> tid : c1 >> (tid - 64)) & 1ull)) s.pos[cuts_upto(c0, c1, tid)] = (unsigned char)tid;
    if (tid == 0) s.pos[0] = 0;
    __syncthreads();
    for (int i = tid; i < kBoundNodes * kBoundEntries; i += kBoundThreads) {
        const int j = i / kBoundEntries, e = i % kBoundEntries;
        uint32_t d = kBoundNone | (kBoundNone << 16);
        if (e <= count) {
            const int end = window_end(s.P, L, (double)s.M[s.node[j]], s.pos[e]);
            const int top = cuts_upto(c0, c1, end);
            if (end == L) {
                d = kBoundEnds | (kBoundEnds << 16);
            } else if (top > e) {
                const int r = 31 - __clz(top - e);
                d = (uint32_t)(r * 256 + (e + 1) * 2) | (uint32_t)(r * 256 + (top - (1 << r) + 1) * 2) << 16;
            }
        }
        s.query[j][e] = d;
        // a set of one node: its segment runs to the end of the chain
        const uint16_t one = (d & 0xFFFFu) == kBoundEnds ? 0 : (uint16_t)kBoundInf;
        reinterpret_cast<uint16_t*>(s.rows)[(int)s.place[1 << j] * kBoundEntries + e] = one;
    }
    for (int i = tid; i < kBoundNodes * kBoundNodes * kBoundEntries; i += kBoundThreads) {
        const int e = i % kBoundEntries, p = i / kBoundEntries, a = p / kBoundNodes, b = p % kBoundNodes;
        uint32_t c = kBoundInf;
        if (a != b && e >= 1 && e <= count) {
            const uint32_t bits = __float_as_uint(__fdiv_rn(s.t[s.pos[e] - 1], s.B[s.node[a] * n + s.node[b]]));
            c = bits >= kInfBits ? kBoundInf : (bits + 0xFFFFu) >> 16;
        }
        s.q[a][b][e] = (uint16_t)c;
    }
    __syncthreads();
    const int most = pmax < kBoundNodes ? pmax : kBoundNodes;   // sets of as many nodes stand for all smaller ones
    if (most > 1) bound_level<1>(s, lane, wave);
    if (most > 2) bound_level<2>(s, lane, wave);
    if (most > 3) bound_level<3>(s, lane, wave);
    if (most > 4) bound_level<4>(s, lane, wave);
    if (most > 5) bound_level<5>(s, lane, wave);
    if (most > 6) bound_level<6>(s, lane, wave);
    if (most > 7) bound_level<7>(s, lane, wave);
    if (most > 8) bound_level<8>(s, lane, wave);
    const uint32_t* rows = s.rows + (most & 1 ? 0 : kBoundOddRows * kBoundRow);
    const int count_rows = (s.level[most + 1] - s.level[most]) * most;
    uint32_t best = kBoundInf;
    for (int i = tid; i < count_rows; i += kBoundThreads) {
        const uint32_t x = rows[i * kBoundRow] & 0xFFFFu;
        best = x < best ? x : best;
    }
    if (best < kBoundInf) atomicMin(&s.best, best);
    __syncthreads();
    if (tid == 0) reinterpret_cast<uint32_t*>(out + (size_t)inst * stride)[blockIdx.x] = s.best << 16;
}

// ---------------------------------------------------------------------------------------------
// Tables of one instance, as cluster_tables_kernel makes them, of the nodes and cuts that can matter; one workgroup.
// ---------------------------------------------------------------------------------------------
namespace {
template <int MAXN>
struct ConfineShared {
    double P[PPO_MAX_L + 64 + 1];
    float t[PPO_MAX_L], m[PPO_MAX_L], M[MAXN], B[MAXN * MAXN];
    unsigned char hi[MAXN][PPO_MAX_L + 4];
    unsigned long long cuts[2];                                    // bit e: the cut e
    unsigned long long link[MAXN][MAXN];                           // by positions, as the following
    unsigned long long ends[MAXN], back[2][MAXN], fore[2][MAXN], reach[MAXN];
    unsigned char top[MAXN][64];                                   // last position inside the window
    unsigned char pos[PPO_MAX_L + 1], node[MAXN], ord[PPO_MAX_L];
    int changed[2][MAXN];
};
// t / B <= bound, and a little more: no quotient whose binary32 value is at most `bound` is missed, and no division is needed.
// A normal quotient is off by 2^-24 of itself.  Below the normal range it is off by up to 2^-150 whatever its size (and t / B
// rounds to 0 for t up to 2^-150 B), so every t / B that is not normal is taken for one within a bound that is not: 2^-126 B.
__device__ __forceinline__ float link_limit(uint32_t bound, float bandwidth) {
    constexpr uint32_t kLeastNormal = 0x00800000u;
    return __uint_as_float(bound > kLeastNormal ? bound : kLeastNormal) * bandwidth * 1.000001f + 1.2e-38f;
}
// all lanes' bits, in all lanes: shifts within rows of 16, then the last lane of a row to the next row, of two rows to the
// next two
__device__ __forceinline__ uint32_t or_lanes(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned long long or_lanes(unsigned long long v) {
    return (unsigned long long)or_lanes((uint32_t)v) | (unsigned long long)or_lanes((uint32_t)(v >> 32)) << 32;
}
// Inputs, prefix sums and windows (hi) of an instance; then, if there is a bound and few enough cuts are within it, the nodes
// and cuts that lie on a walk of up to `rounds` segments: true.  All threads of the workgroup, in step.
template <int MAXN>
__device__ __forceinline__ bool confine(ConfineShared<MAXN>& s, const float* __restrict__ t, const float* __restrict__ m,
                                        const float* __restrict__ M, const float* __restrict__ B, int L, int n, int rounds, int inst,
                                        uint32_t bound, unsigned long long& cuts0, unsigned long long& cuts1, unsigned long long& nodes) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = kClPreThreads / 64;
    if (tid < L) {
        const float x = t[(size_t)inst * L + tid];
        s.t[tid] = x == 0.0f ? 0.0f : x;   // -0 is a size of zero: +0
        s.m[tid] = m[(size_t)inst * L + tid];
    }
    if (tid < n) s.M[tid] = M[(size_t)inst * n + tid];
    for (int i = tid; i < n * n; i += kClPreThreads) {
        const int a = i / n, b = i - a * n;   // the element with the smaller row index is the one read
        s.B[i] = B[(size_t)inst * n * n + (a < b ? i : b * n + a)];
    }
    __syncthreads();
    if (wave == 0) prefix_sums(s.m, L, lane, s.P);
    if (wave == 1) {
        // cuts with a link of at most the bound: over the fastest link
        float most = 0.0f;
        for (int i = lane; i < n * n; i += 64) most = i / n != i % n && s.B[i] > most ? s.B[i] : most;
        for (int off = 32; off >= 1; off >>= 1) {
            const float o = __shfl_xor(most, off, 64);
            most = o > most ? o : most;
        }
        const float limit = link_limit(bound, most);
        for (int h = 0; h < 2; ++h) {
            const int e = lane + 64 * h;
            const bool in = e >= 1 && e < L && s.t[e >= 1 && e < L ? e - 1 : 0] <= limit;
            const unsigned long long some = __ballot(in);
            if (lane == 0) s.cuts[h] = some;
        }
    }
    __syncthreads();
    for (int i = tid; i < n * (L + 1); i += kClPreThreads) {
        const int j = i / (L + 1), e = i - j * (L + 1);
        s.hi[j][e] = (unsigned char)window_end(s.P, L, (double)s.M[j], e);
    }
    const unsigned long long c0 = s.cuts[0], c1 = s.cuts[1];
    const int count = __popcll(c0) + __popcll(c1);
    if (bound >= kInfBits || count > kMostCuts) return false;
    {
        // positions: 0 the start of the chain, then the cuts
        if (tid >= 1 && tid < L && ((tid < 64 ? c0 >> tid : c1 >> (tid - 64)) & 1ull)) s.pos[cuts_upto(c0, c1, tid)] = (unsigned char)tid;
        if (tid == 0) s.pos[0] = 0;
        if (tid < 2 * MAXN) s.changed[tid / MAXN][tid % MAXN] = 0;   // one for every round
        __syncthreads();
        const bool is_cut = lane >= 1 && lane <= count;
        const float size = s.t[is_cut ? s.pos[lane] - 1 : 0];
        for (int a = wave; a < n; a += waves)
            for (int b = a; b < n; ++b) {
                const unsigned long long some = a < b ? __ballot(is_cut && size <= link_limit(bound, s.B[a * n + b])) : 0ull;
                if (lane == 0) s.link[a][b] = s.link[b][a] = some;
            }
        for (int j = wave; j < n; j += waves) {
            const int end = lane <= count ? (int)s.hi[j][s.pos[lane <= count ? lane : 0]] : 0;
            const unsigned long long ends = __ballot(lane <= count && end == L);
            s.top[j][lane] = (unsigned char)(lane <= count ? cuts_upto(c0, c1, end < L - 1 ? end : L - 1) : 0);
            if (lane == 0) {
                s.ends[j] = s.back[0][j] = ends;
                s.fore[0][j] = 1ull;
            }
        }
        __syncthreads();
        // a placement has at most that many segments: as many rounds find every cut that matters
        int now = 0;
        for (int round = 0; round < rounds; ++round) {
            for (int j = wave; j < n; j += waves) {
                const unsigned long long rest = or_lanes(lane < n ? s.link[j][lane < n ? lane : 0] & s.back[now][lane < n ? lane : 0] : 0ull);
                // a start whose window holds a cut from which it goes on
                const int top = s.top[j][lane];
                const unsigned long long window = top > lane ? ((top >= 63 ? 0ull : 1ull << (top + 1)) - 1ull) & ~((2ull << lane) - 1ull) : 0ull;
                const unsigned long long some = __ballot(lane <= count && (window & rest) != 0ull) | s.ends[j];
                if (lane == 0) {
                    s.back[now ^ 1][j] = some;
                    if (some != s.back[now][j]) s.changed[0][round] = 1;
                }
            }
            __syncthreads();
            now ^= 1;
            if (!s.changed[0][round]) break;
        }
        const int done = now;
        now = 0;
        for (int round = 0; round < rounds; ++round) {
            for (int j = wave; j < n; j += waves) {
                // cuts that a window starting in fore & back covers: the latest start before a cut decides
                const unsigned long long start = s.fore[now][j] & s.back[done][j], before = start & ((1ull << lane) - 1ull);
                const int latest = before ? 63 - __clzll((long long)before) : 0;
                const unsigned long long some = __ballot(lane <= count && before && (int)s.top[j][latest] >= lane);
                if (lane == 0) s.reach[j] = some;
            }
            __syncthreads();
            for (int j = wave; j < n; j += waves) {
                const unsigned long long come = or_lanes(lane < n ? s.link[lane < n ? lane : 0][j] & s.reach[lane < n ? lane : 0] : 0ull);
                if (lane == 0) {
                    const unsigned long long some = s.fore[now][j] | come;
                    s.fore[now ^ 1][j] = some;
                    if (some != s.fore[now][j]) s.changed[1][round] = 1;
                }
            }
            __syncthreads();
            now ^= 1;
            if (!s.changed[1][round]) break;
        }
        const unsigned long long mine = lane < n ? s.fore[now][lane < n ? lane : 0] & s.back[done][lane < n ? lane : 0] : 0ull;
        const unsigned long long left = __ballot(mine != 0ull);
        const unsigned long long at = or_lanes(mine);
        // back to cuts: position i is the i-th one
        const int e0 = lane, e1 = lane + 64;
        const bool k0 = ((c0 >> lane) & 1ull) && ((at >> cuts_upto(c0, c1, e0)) & 1ull);
        const bool k1 = ((c1 >> lane) & 1ull) && ((at >> cuts_upto(c0, c1, e1)) & 1ull);
        const unsigned long long n0 = __ballot(k0), n1 = __ballot(k1);
        __syncthreads();
        cuts0 = n0;
        cuts1 = n1;
        nodes = left;
        return left != 0ull;
    }
}
}  // namespace

__global__ __launch_bounds__(kClPreThreads) void cluster_reduce_kernel(const float* __restrict__ t, const float* __restrict__ m,
                                                                      const float* __restrict__ M, const float* __restrict__ B,
                                                                      ClusterLayout whole, unsigned char* __restrict__ ws) {
    __shared__ ConfineShared<PPO_CLUSTER_MAX_N> s;
    const int L = whole.L, n = whole.n, inst = blockIdx.x, tid = threadIdx.x;
    unsigned char* base = ws + (size_t)inst * whole.stride;
    const uint32_t* bounds = reinterpret_cast<const uint32_t*>(base + whole.img_off);
    const uint32_t u0 = bounds[0], u1 = bounds[1];
    unsigned long long c0 = 0ull, c1 = 0ull, left = 0ull;
    bool reduced = confine(s, t, m, M, B, L, n, n, inst, u0 < u1 ? u0 : u1, c0, c1, left);
    __syncthreads();
    if (reduced) {
        // the smaller tables leave room for the record, and with the binomial coefficients take no more LDS than the levels are given
        const ClusterLayout y2 = ClusterLayout::make(__popcll(c0) + __popcll(c1) + 1, __popcll(left));
        reduced = y2.stride <= whole.record_off() &&
                  y2.q_image_bytes() + y2.query_bytes() + kClBinomialBytes <= whole.q_image_bytes() + whole.query_bytes();
    }
    const uint32_t nodes = reduced ? (uint32_t)left : (1u << n) - 1u;
    if (!reduced) {   // every cut
        c0 = (L >= 64 ? ~0ull : (1ull << L) - 1ull) & ~1ull;
        c1 = L <= 64 ? 0ull : L >= 128 ? ~0ull : (1ull << (L - 64)) - 1ull;
    }
    const ClusterLayout y = reduced ? ClusterLayout::make(__popcll(c0) + __popcll(c1) + 1, __popc(nodes)) : whole;
    if (tid == 0) {
        *reinterpret_cast<uint32_t*>(base + whole.flag_off()) = reduced ? 1u : 0u;
        if (reduced) {
            ClusterRecord* r = reinterpret_cast<ClusterRecord*>(base + whole.record_off());
            r->cuts[0] = c0;
            r->cuts[1] = c1;
            r->nodes = nodes;
        }
    }
    // from here on as without a bound, by position and by place among the nodes left
    if (tid >= 1 && tid < L && ((tid < 64 ? c0 >> tid : c1 >> (tid - 64)) & 1ull)) s.pos[cuts_upto(c0, c1, tid)] = (unsigned char)tid;
    if (tid == 0) {
        s.pos[0] = 0;
        s.pos[y.L] = (unsigned char)L;
    }
    if (tid < n && ((nodes >> tid) & 1u)) s.node[__popc(nodes & ((1u << tid) - 1u))] = (unsigned char)tid;
    __syncthreads();
    for (int i = tid; i < y.n * (y.L + 1); i += kClPreThreads) {
        const int j = i / (y.L + 1), e = i - j * (y.L + 1), end = s.hi[s.node[j]][s.pos[e]];
        base[y.hi_off + i] = (unsigned char)(end == L ? y.L : cuts_upto(c0, c1, end));
    }
    // each link's quotients in the order of t (see cluster_tables_kernel)
    for (int i = tid; i < y.L - 1; i += kClPreThreads) {
        const float x = s.t[s.pos[i + 1] - 1];
        int place = 0;
        for (int i2 = 0; i2 < y.L - 1; ++i2) {
            const float x2 = s.t[s.pos[i2 + 1] - 1];
            place += (x2 < x || (x2 == x && i2 < i)) ? 1 : 0;
        }
        s.ord[place] = (unsigned char)i;
        base[y.ord_off + place] = (unsigned char)i;
    }
    __syncthreads();
    float* qv = reinterpret_cast<float*>(base + y.qv_off);
    if (tid == 0) reinterpret_cast<float*>(base + y.dec_off)[0] = 0.0f;
    for (int i = tid; i < y.nq; i += kClPreThreads) {
        const int p = i / (y.L - 1), r = i - p * (y.L - 1);
        int a = 0, rem = p;
        while (rem >= y.n - 1 - a) { rem -= y.n - 1 - a; ++a; }
        qv[i] = __fdiv_rn(s.t[s.pos[s.ord[r] + 1] - 1], s.B[s.node[a] * n + s.node[a + 1 + rem]]);
    }
}

// Nodes and cuts of an instance of the search for few segments (ppo_cluster_few.hip), which makes its tables of them.
__global__ __launch_bounds__(kClPreThreads) void few_confine_kernel(const float* __restrict__ t, const float* __restrict__ m,
                                                                   const float* __restrict__ M, const float* __restrict__ B, int L,
                                                                   int n, int pmax, FewConfined* __restrict__ out, size_t stride) {
    extern __shared__ __align__(16) unsigned char bound_sm[];
    ConfineShared<PPO_CLUSTER_FEW_MAX_N>& s = *reinterpret_cast<ConfineShared<PPO_CLUSTER_FEW_MAX_N>*>(bound_sm);
    FewConfined* mine = reinterpret_cast<FewConfined*>(reinterpret_cast<unsigned char*>(out) + (size_t)blockIdx.x * stride);
    const uint32_t u0 = mine->bounds[0], u1 = mine->bounds[1];
    unsigned long long c0 = 0ull, c1 = 0ull, left = 0ull;
    const uint32_t bound = u0 < u1 ? u0 : u1;
    const bool in = bound < kInfBits && confine(s, t, m, M, B, L, n, pmax, (int)blockIdx.x, bound, c0, c1, left);
    __syncthreads();   // (the bounds lie where the nodes go)
    if (threadIdx.x == 0) {
        mine->in = in ? 1u : 0u;
        mine->bound = bound;
        mine->nodes = left;
        mine->cuts[0] = c0;
        mine->cuts[1] = c1;
    }
}

static hipError_t launch_bound(const float* t, const float* m, const float* M, const float* B, int L, int n, int pmax, int n_inst,
                               unsigned char* out, size_t stride, hipStream_t stream) {
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&cluster_bound_kernel), lds_allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cluster_bound_kernel, dim3(2, n_inst), dim3(kBoundThreads), sizeof(BoundShared), stream, t, m, M, B, L, n, pmax,
                       out, stride);
    return hipGetLastError();
}

hipError_t launch_cluster_reduce(const float* t, const float* m, const float* M, const float* B, const ClusterLayout& y, int n_inst,
                                 unsigned char* ws, hipStream_t stream) {
    const hipError_t e = launch_bound(t, m, M, B, y.L, y.n, y.n, n_inst, ws + y.img_off, y.stride, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cluster_reduce_kernel, dim3(n_inst), dim3(kClPreThreads), 0, stream, t, m, M, B, y, ws);
    return hipGetLastError();
}

hipError_t launch_few_confine(const float* t, const float* m, const float* M, const float* B, int L, int n, int pmax, int n_inst,
                              FewConfined* out, size_t stride, hipStream_t stream) {
    hipError_t e = launch_bound(t, m, M, B, L, n, pmax, n_inst, reinterpret_cast<unsigned char*>(out), stride, stream);
    if (e != hipSuccess) return e;
    static std::atomic<uint64_t> lds_allowed{0};
    e = allow_full_lds(reinterpret_cast<const void*>(&few_confine_kernel), lds_allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(few_confine_kernel, dim3(n_inst), dim3(kClPreThreads), sizeof(ConfineShared<PPO_CLUSTER_FEW_MAX_N>), stream, t, m,
                       M, B, L, n, pmax, out, stride);
    return hipGetLastError();
}

}  // namespace ppo
