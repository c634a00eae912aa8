// The paper's own placement algorithm, for scoring against the exact optimum: partitioning, classes, matching and the
// bottleneck of the result in one launch, one workgroup per instance.
//
// Sec. III-B2: the cuts come from the partitioning step (Alg. 1, ppo_partition.h); their transfer sizes are sorted into
// classes (Eq. 5); classes are matched from the highest down, within a class the runs of consecutive cuts from the
// longest down (Alg. 3); a run of r cuts gets a path of r + 1 nodes of the communication graph whose weakest link is as
// strong as possible: bisection over the descending list of bandwidths for the highest threshold at which the graph of
// links at or above it (Eq. 8) still holds such a path between the ends that neighbouring runs have fixed (Alg. 2).
//
// Readings (the paper leaves them open): classes are bins of equal width between the least and the greatest transfer size
// of the chain's candidate cuts; the path search, colour coding in the paper, is a depth-first search in increasing node
// order that returns the smallest sequence and gives up after kPathBudget nodes put on the path; if a run cannot be
// matched, the matching is tried again with one class fewer.
//
// 50 instances of 50 nodes, 50 layers: 1530 us -> 72 us per call (one lane searching on memory, the partitioning step a
// launch of its own); 4096 of them: 4.96 ms -> 0.47 ms.
//
// The result is defined by sequential searches, so latency bounds it: what is left is to make each step short.
//   - Bandwidths are sorted once; from then on a link is its place among the distinct bandwidths, 16 bits, and lane a
//     keeps node a's row of them in 32 registers: the masks of a threshold are 4 instructions per 2 links.
//   - A search keeps its path and the candidates left at every position in lanes, and settles the last three positions
//     of a path with one step over all lanes (kpath_search): a path search of depth d costs what its first d - 3
//     positions cost, while the budget is counted as if every node had been put on the path.
//   - 2^DEPTH waves bisect DEPTH steps at a time: each wave searches at one of the thresholds that these steps can come
//     to, then all follow the outcomes.  A wave whose threshold cannot be come to any more gives up.
#include "ppo_partition.h"

namespace ppo {

constexpr int kKpathMaxN = PPO_HEURISTIC_MAX_N;
constexpr int kKpathMaxPairs = kKpathMaxN * (kKpathMaxN - 1) / 2;
constexpr int kKpathSort = 2048;           // power of two that holds every pair
constexpr int kKpathPitch = 72;            // halfwords per row of places: 16-byte aligned rows on different banks
constexpr uint32_t kKpathBudget = 20000u;
constexpr uint32_t kNoLink = 0x7FFFu;      // beyond every place; a difference of two places keeps its sign in 16 bits
static_assert(kKpathMaxPairs <= kKpathSort && kKpathSort / 32 <= 64 && kKpathMaxN == 64, "one lane per node and per word of places");

typedef short kp_short2 __attribute__((ext_vector_type(2)));

struct KpathShared {
    unsigned long long key[kKpathSort];               // (descending bandwidth, pair)
    float value[kKpathSort];                          // the distinct bandwidths, descending
    alignas(16) uint16_t place[kKpathMaxN][kKpathPitch];   // of link (a, b) at [a][2 (b mod 32) + b / 32]
    uint32_t listed[3][kKpathSort / 32];              // places of the links among the nodes of a run, one bit each
    uint32_t needless[3];                             // thresholds of a round that the bisection cannot come to
    uint32_t chunk_count[kKpathSort / 64];
    unsigned char outcome[3][16];
    unsigned char path[3][16][kKpathMaxN];
    float t[PPO_MAX_L];
    PartitionShared part;
    int segs, one_way;
};

__device__ __forceinline__ int kpath_slot(int b) { return 2 * (b & 31) + (b >> 5); }

// Depth-first search for the smallest sequence of k >= 2 distinct nodes: first `start` and last `end` where given (>= 0),
// every other one from `avail`, consecutive ones linked: lane v holds the nodes that v is linked to (adj) and those linked
// to v (adj_in).  On success lane i of `path` holds the node at position i.  `needless` is looked at now and then: once
// its bit `bit` is set the result is not asked for (returns false).  Ends: every node put on the path, and every step
// over the last three positions but an empty one, takes from the budget.
__device__ __forceinline__ bool kpath_search(unsigned long long adj, unsigned long long adj_in, unsigned long long avail, int k,
                                             int start, int end, int lane, volatile uint32_t* needless, uint32_t bit, int& path) {
    const unsigned long long first_set = start >= 0 ? 1ull << start : avail;
    const unsigned long long last_set = end >= 0 ? 1ull << end : avail;
    if (k == 2) {   // never more than 65 nodes put on the path
        const unsigned long long nb = adj & last_set;
        const unsigned long long ok = __ballot(nb != 0ull) & first_set;
        if (!ok) return false;
        const int v = __ffsll((long long)ok) - 1;
        const int w = __ffsll((long long)readlane_u64(nb, v)) - 1;
        path = lane == 0 ? v : w;
        return true;
    }
    uint32_t budget = kKpathBudget, look = 0;
    unsigned long long on_path = 0ull, left = first_set;   // left: candidates not yet tried at this position
    uint32_t left_lo = 0, left_hi = 0;                     // lane i: those of position i
    int pos = 0;
    for (;;) {
        if (pos == k - 3 && left) {
            // Lane v stands for v at this position, its neighbours u for the next, theirs for the last.  A u can be
            // followed unless v is the only node that it could be followed by.
            const unsigned long long last = last_set & ~on_path;
            const unsigned long long nb = adj & last;
            const int cnt = __popcll(nb);
            const unsigned long long one = __ballot(cnt == 1), more = __ballot(cnt >= 2);
            const unsigned long long mid = adj & avail & ~on_path;
            const unsigned long long into = ((last >> lane) & 1ull) ? adj_in : 0ull;
            const unsigned long long good = mid & (more | (one & ~into));
            // nodes that the search puts on the path from v on: v, every u up to the first good one, the last node
            const uint32_t cost = good ? 2u + (uint32_t)__popcll(mid & (good ^ (good - 1ull))) : 1u + (uint32_t)__popcll(mid);
            const unsigned long long found = __ballot(good != 0ull) & left;
            const unsigned long long tried = found ? left & (found ^ (found - 1ull)) : left;
            uint32_t spent = 0;
#pragma unroll
            for (int b = 0; b < 7; ++b) spent += (uint32_t)__popcll(__ballot((cost >> b) & 1u) & tried) << b;
            if (spent > budget) return false;
            if (found) {
                const int v = __ffsll((long long)found) - 1;
                const int u = __ffsll((long long)readlane_u64(good, v)) - 1;
                const int w = __ffsll((long long)(readlane_u64(nb, u) & ~(1ull << v))) - 1;
                if (lane == pos) path = v;
                if (lane == pos + 1) path = u;
                if (lane == pos + 2) path = w;
                return true;
            }
            budget -= spent;
            left = 0ull;
        }
        if ((++look & 31u) == 0u && ((uint32_t)__builtin_amdgcn_readfirstlane((int)*needless) >> bit & 1u)) return false;
        if (left) {
            if (budget == 0u) return false;
            --budget;
            const int v = __ffsll((long long)left) - 1;
            left &= left - 1ull;
            if (lane == pos) {
                path = v;
                left_lo = (uint32_t)left;
                left_hi = (uint32_t)(left >> 32);
            }
            on_path |= 1ull << v;
            ++pos;
            left = readlane_u64(adj, v) & avail & ~on_path;
        } else {
            if (pos == 0) return false;
            --pos;
            on_path &= ~(1ull << __builtin_amdgcn_readlane(path, pos));
            left = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)left_hi, pos) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)left_lo, pos);
        }
    }
}

template <int DEPTH>
__global__ __launch_bounds__(64 << DEPTH) void kpath_kernel(const float* __restrict__ t, const float* __restrict__ m, int L,
                                                            const float* __restrict__ kappa, const float* __restrict__ B_all,
                                                            int n, int n_classes, float* __restrict__ beta_out,
                                                            int32_t* __restrict__ segs_out, int32_t* __restrict__ cuts_out,
                                                            int32_t* __restrict__ order_out, int32_t* __restrict__ classes_out) {
    constexpr int kThreads = 64 << DEPTH, kWaves = 1 << DEPTH;
    __shared__ KpathShared S;
    const int inst = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* ti = t + (size_t)inst * L;
    const float* B = B_all + (size_t)inst * n * n;
    const int pairs = n * (n - 1) / 2;
    int sort = 64;
    while (sort < pairs) sort <<= 1;

    // ---- the cuts (wave 0), the keys of all links a < b, tables cleared
    if (wave == 0) {
        double sum;
        const int segs = min_sum_partition_wave(ti, m + (size_t)inst * L, L, (double)kappa[inst], lane, S.part, sum);
        if (lane == 0) {
            S.segs = segs;
            S.one_way = 0;
        }
        if (lane < 3) S.needless[lane] = 0u;
    }
    for (int i = tid; i < L; i += kThreads) S.t[i] = ti[i];
    for (int i = tid; i < kKpathMaxN * kKpathPitch / 2; i += kThreads) reinterpret_cast<uint32_t*>(S.place)[i] = kNoLink | (kNoLink << 16);
    for (int i = tid; i < 3 * (kKpathSort / 32); i += kThreads) (&S.listed[0][0])[i] = 0u;
    for (int i = pairs + tid; i < sort; i += kThreads) S.key[i] = ~0ull;
    bool differs = false;
    for (int i = tid; i < n * n; i += kThreads) {
        const int a = i / n, b = i - a * n;
        if (a >= b) continue;
        const uint32_t bits = __float_as_uint(B[i]);
        differs |= bits != __float_as_uint(B[b * n + a]);
        const uint32_t rising = bits ^ ((bits >> 31) ? 0xFFFFFFFFu : 0x80000000u);
        S.key[a * (2 * n - a - 1) / 2 + b - a - 1] = ((unsigned long long)~rising << 32) | (uint32_t)(a | (b << 8));
    }
    __syncthreads();
    if (differs) S.one_way = 1;
    const int p = S.segs;
    int32_t* cuts_o = cuts_out + (size_t)inst * (L > 1 ? L - 1 : 0);
    int32_t* order_o = order_out + (size_t)inst * n;
    auto fail = [&]() {
        for (int i = tid; i < L - 1; i += kThreads) cuts_o[i] = -1;
        for (int i = tid; i < n; i += kThreads) order_o[i] = -1;
        if (tid == 0) {
            beta_out[inst] = __uint_as_float(kInfBits);
            segs_out[inst] = 0;
            if (classes_out) classes_out[inst] = 0;
        }
    };
    if (p == 0 || p > n) { fail(); return; }

    // ---- links in descending order of bandwidth.  64 pairs of elements a stride of at most 64 apart are one wave's.
    for (int size = 2; size <= sort; size <<= 1)
        for (int j = size >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < sort / 2; i += kThreads) {
                const int x = 2 * i - (i & (j - 1)), y = x + j;
                const unsigned long long u = S.key[x], v = S.key[y];
                if ((u > v) == ((x & size) == 0)) {
                    S.key[x] = v;
                    S.key[y] = u;
                }
            }
            const int next = j > 1 ? j >> 1 : size;
            if (j > 64 || next > 64) __syncthreads(); else wave_lds_fence();
        }
    __syncthreads();
    auto value_of = [](unsigned long long key) -> float {
        const uint32_t rising = ~(uint32_t)(key >> 32);
        return __uint_as_float(rising ^ ((rising >> 31) ? 0x80000000u : 0xFFFFFFFFu));
    };
    auto differs_from_last = [&](int i) -> bool {
        return i < pairs && (i == 0 || value_of(S.key[i]) != value_of(S.key[i - 1]));
    };
    const int chunks = sort / 64;
    for (int c = wave; c < chunks; c += kWaves) {
        const unsigned long long heads = __ballot(differs_from_last(c * 64 + lane));
        if (lane == 0) S.chunk_count[c] = (uint32_t)__popcll(heads);
    }
    __syncthreads();
    int distinct = 0;
    {
        const uint32_t count = lane < chunks ? S.chunk_count[lane] : 0u;
        uint32_t upto = count;
        for (int off = 1; off < 32; off <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)upto, off, 64);
            if (lane >= off) upto += o;
        }
        distinct = __builtin_amdgcn_readlane((int)upto, chunks - 1);
        for (int c = wave; c < chunks; c += kWaves) {
            const int i = c * 64 + lane;
            const bool head = differs_from_last(i);
            const unsigned long long heads = __ballot(head);
            const int before = __builtin_amdgcn_readlane((int)(upto - count), c);
            const int place = before + __popcll(heads & (~0ull >> (63 - lane))) - 1;
            if (i < pairs) {
                const unsigned long long key = S.key[i];
                const int a = (int)(key & 0xFFu), b = (int)((key >> 8) & 0xFFu);
                S.place[a][kpath_slot(b)] = (uint16_t)place;
                S.place[b][kpath_slot(a)] = (uint16_t)place;
                if (head) S.value[place] = value_of(key);
            }
        }
    }
    __syncthreads();
    const bool one_way = S.one_way != 0;
    if (one_way) {
        // a link whose two directions differ: thresholds are taken from a < b, the other direction is placed among them
        for (int i = tid; i < n * n; i += kThreads) {
            const int a = i / n, b = i - a * n;
            if (a <= b || __float_as_uint(B[i]) == __float_as_uint(B[b * n + a])) continue;
            const float x = B[i];
            int lo = 0, hi = distinct;   // first distinct bandwidth that x reaches
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (x >= S.value[mid]) hi = mid; else lo = mid + 1;
            }
            S.place[a][kpath_slot(b)] = (uint16_t)(lo < distinct ? (uint32_t)lo : kNoLink);
        }
        __syncthreads();
    }
    uint32_t row[32];   // of node `lane`: places of its links to node i (low half) and i + 32
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint4 v = reinterpret_cast<const uint4*>(S.place[lane])[i];
        row[4 * i] = v.x;
        row[4 * i + 1] = v.y;
        row[4 * i + 2] = v.z;
        row[4 * i + 3] = v.w;
    }

    // ---- Eq. 5 classes, then Alg. 3, with fewer classes if a run cannot be matched.  Every wave does the same steps:
    // lane i stands for cut i and segment i (p <= n <= 64).
    float lo = S.t[0], hi = lo;
    for (int i = lane; i < L - 1; i += 64) {
        const float x = S.t[i];
        lo = x < lo ? x : lo;
        hi = x > hi ? x : hi;
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const float a = __shfl_xor(lo, off, 64), b = __shfl_xor(hi, off, 64);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    const bool is_cut = lane + 1 < p;
    const int my_cut = is_cut ? (int)S.part.cut[lane] : 0;
    const float my_size = is_cut ? S.t[my_cut - 1] : 0.0f;
    int my_node = -1;   // node of segment `lane`, -1 while open
    int used = 0, run_count = 0, round = 0;
    if (p == 1) {
        my_node = 0;
        used = n_classes;
    }
    for (int nc = n_classes; nc >= 1 && !used; --nc) {
        int cls = nc - 1;
        if (hi != lo) {
            const double x = floor(((double)my_size - (double)lo) / ((double)hi - (double)lo) * (double)nc);
            cls = x < (double)(nc - 1) ? (int)x : nc - 1;
        }
        // runs of cuts of one class, in the order of matching: higher class, longer, earlier
        const int cls_before = __shfl_up(cls, 1, 64);
        const unsigned long long heads = __ballot(is_cut && (lane == 0 || cls != cls_before));
        const unsigned long long after = lane < 63 ? heads >> (lane + 1) : 0ull;
        const int my_len = after ? __ffsll((long long)after) : p - 1 - lane;
        const int runs = __popcll(heads);
        int my_turn = 0;
        for (unsigned long long hb = heads; hb; hb &= hb - 1ull) {
            const int o = __ffsll((long long)hb) - 1;
            const int oc = __builtin_amdgcn_readlane(cls, o), ol = __builtin_amdgcn_readlane(my_len, o);
            my_turn += (oc > cls || (oc == cls && (ol > my_len || (ol == my_len && o < lane)))) ? 1 : 0;
        }
        my_node = -1;
        unsigned long long avail = n < 64 ? (1ull << n) - 1ull : ~0ull;
        bool ok = true;
        for (int r = 0; r < runs && ok; ++r) {
            const int first = __ffsll((long long)(__ballot(my_turn == r) & heads)) - 1;
            const int len = __builtin_amdgcn_readlane(my_len, first);
            const int start = __builtin_amdgcn_readlane(my_node, first), end = __builtin_amdgcn_readlane(my_node, first + len);
            if (start >= 0 && end >= 0 && len == 1) continue;
            const int k = len + 1;
            // the distinct bandwidths among the nodes of this run; the list after the next is cleared for it
            unsigned long long nodes = avail;
            if (start >= 0) nodes |= 1ull << start;
            if (end >= 0) nodes |= 1ull << end;
            const int list = run_count % 3;
            ++run_count;
            if (tid < kKpathSort / 32) S.listed[run_count % 3][tid] = 0u;
            for (int i = tid; i < n * 64; i += kThreads) {
                const int a = i >> 6, b = i & 63;
                if (a < b && ((nodes >> a) & 1ull) && ((nodes >> b) & 1ull)) {
                    const uint32_t x = S.place[a][kpath_slot(b)];
                    if (x < (uint32_t)kKpathSort) atomicOr(&S.listed[list][x >> 5], 1u << (x & 31u));
                }
            }
            __syncthreads();
            const uint32_t word = S.listed[list][lane];
            int upto = __popc(word);
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(upto, off, 64);
                if (lane >= off) upto += o;
            }
            const int before = upto - __popc(word);
            // Alg. 2: bisection, DEPTH steps a round; thresholds of a round are numbered like a heap
            int low = 0, high = __builtin_amdgcn_readlane(upto, 63);
            bool found = false;
            int best_path = 0;
            for (; low < high; ++round) {
                const int slot = round % 3;
                if (tid == 0) S.needless[(round + 1) % 3] = 0u;
                if (wave >= 1) {
                    int l = low, h = high;
                    for (int b = 30 - __builtin_clz((unsigned)wave); b >= 0 && l < h; --b) {
                        const int median = (l + h) / 2;
                        if ((wave >> b) & 1) l = median + 1; else h = median;
                    }
                    if (l < h) {
                        const int median = (l + h) / 2;
                        const int at = __ffsll((long long)__ballot(before <= median && median < upto)) - 1;
                        uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)word, at);
                        for (int skip = median - __builtin_amdgcn_readlane(before, at); skip > 0; --skip) w &= w - 1u;
                        const uint32_t place = (uint32_t)at * 32u + (uint32_t)__ffs(w) - 1u;
                        const uint32_t place2 = place | (place << 16);
                        uint32_t none_lo = 0, none_hi = 0;   // nodes that `lane` is not linked to: places beyond this one
#pragma unroll
                        for (int i = 31; i >= 0; --i) {
                            const uint32_t d = __builtin_bit_cast(uint32_t, (kp_short2)(__builtin_bit_cast(kp_short2, place2) -
                                                                                       __builtin_bit_cast(kp_short2, row[i])));
                            none_hi = __builtin_amdgcn_alignbit(none_hi, d, 31);
                            none_lo = __builtin_amdgcn_alignbit(none_lo, d << 16, 31);
                        }
                        const unsigned long long adj = ~(((unsigned long long)none_hi << 32) | none_lo);
                        unsigned long long adj_in = adj;
                        if (one_way) {
                            for (int b = 0; b < 64; ++b) {
                                const unsigned long long in = __ballot((adj >> b) & 1ull);
                                if (lane == b) adj_in = in;
                            }
                        }
                        int path = 0;
                        const bool hit = kpath_search(adj, adj_in, avail, k, start, end, lane, &S.needless[slot], (uint32_t)wave, path);
                        if (lane < k) S.path[slot][wave][lane] = (unsigned char)path;
                        if (lane == 0) {
                            S.outcome[slot][wave] = hit ? 1 : 0;
                            const int c = hit ? 2 * wave + 1 : 2 * wave;   // the half that the bisection leaves
                            uint32_t off = 0;
                            for (int s = c, w2 = 1; s < kWaves; s *= 2, w2 *= 2) off |= ((1u << w2) - 1u) << s;
                            if (off) atomicOr(&S.needless[slot], off);
                        }
                    }
                }
                __syncthreads();
                for (int d = 0, node = 1; d < DEPTH && low < high; ++d) {
                    const int median = (low + high) / 2;
                    if (__builtin_amdgcn_readfirstlane((int)S.outcome[slot][node])) {
                        high = median;
                        best_path = S.path[slot][node][lane];
                        found = true;
                        node = 2 * node;
                    } else {
                        low = median + 1;
                        node = 2 * node + 1;
                    }
                }
            }
            if (!found) {
                ok = false;
            } else {
                const int mine = __shfl(best_path, lane >= first ? lane - first : 0, 64);
                if (lane >= first && lane <= first + len) my_node = mine;
                for (int i = 0; i < k; ++i) avail &= ~(1ull << __builtin_amdgcn_readlane(best_path, i));
            }
        }
        if (ok) used = nc;
    }
    if (!used) { fail(); return; }

    // ---- Eq. 2, Eq. 3 of the placement found
    if (wave != 0) return;
    const int next_node = __shfl_down(my_node, 1, 64);
    float gamma = 0.0f;
    if (is_cut) {
        gamma = __fdiv_rn(my_size, B[my_node * n + next_node]);
        gamma = gamma > 0.0f ? gamma : 0.0f;
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const float o = __shfl_xor(gamma, off, 64);
        gamma = o > gamma ? o : gamma;
    }
    for (int i = lane; i < L - 1; i += 64) cuts_o[i] = i + 1 < p ? (int32_t)S.part.cut[i] : -1;
    if (lane < n) order_o[lane] = lane < p ? my_node : -1;
    if (lane == 0) {
        beta_out[inst] = gamma;
        segs_out[inst] = p;
        if (classes_out) classes_out[inst] = used;
    }
}

hipError_t launch_kpath(const float* t, const float* m, int L, const float* kappa, const float* B, int n, int n_inst,
                        int n_classes, float* beta_out, int32_t* segs_out, int32_t* cuts_out, int32_t* order_out,
                        int32_t* classes_out, hipStream_t stream) {
    // 15 thresholds a round for 4 steps of the bisection pay while instances leave compute units idle; beyond one
    // workgroup per compute unit 3 thresholds for 2 steps do less in vain (512 instances of 50 nodes: 143 us with 16 waves
    // each, 108 us with 4)
    if (n_inst <= 256)
        hipLaunchKernelGGL(kpath_kernel<4>, dim3(n_inst), dim3(1024), 0, stream, t, m, L, kappa, B, n, n_classes, beta_out,
                           segs_out, cuts_out, order_out, classes_out);
    else
        hipLaunchKernelGGL(kpath_kernel<2>, dim3(n_inst), dim3(256), 0, stream, t, m, L, kappa, B, n, n_classes, beta_out,
                           segs_out, cuts_out, order_out, classes_out);
    return hipGetLastError();
}

}  // namespace ppo
