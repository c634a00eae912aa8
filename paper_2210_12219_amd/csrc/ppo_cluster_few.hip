// Cluster form of the exact search for LARGE clusters and FEW segments: the hosting nodes are a sequence of
// p <= pmax distinct nodes out of n <= 64 (the paper's evaluation, Sec. IV, uses 5 to 50 devices, and its
// partitioner yields a handful of partitions).  The dynamic programme over sets of UNUSED nodes (ppo_cluster.hip)
// keeps n 2^(n-1) rows and stops at n = 20; here the rows are indexed by the set S of nodes still TO BE used:
//     G[S][j][e] = least bottleneck (Eq. 2) of layers [e, L) when node j (in S) takes the segment that starts at
//                  e and every other node of S takes exactly one of the segments after it
//     G[{j}][j][e] = 0 if layers [e, L) fit node j, else +inf
//     G[S][j][e]   = min over e' in (e, hi_j(e)], e' < L, and j'' in S \ j of max(q_{j,j''}[e'-1], G[S \ j][j''][e'])
// (q_{a,b}[i] = t[i] / B[a][b], Eq. 3; hi_j(e) = last end of a segment from e that fits node j), and
// beta* = min over |S| <= pmax, j in S of G[S][j][0]: sum over c <= pmax of C(n, c) c rows (11.6 million at n = 50,
// pmax = 5).  Values are binary32 bit patterns (non-negative, so they order as unsigned integers): with up to
// 2016 links there are more distinct quotients than 16-bit codes.  Level c = |S| is one launch; the unit of a
// wave is a set S' of c - 1 nodes, whose rows it loads once and extends by every node outside it.  Of the last
// level nothing is kept but the least G[S][j][0] of every node j (all that beta* and the first position of the answer
// need), which lets most of it go unevaluated (few_top_kernel).
// The lexicographically smallest optimal sequence (a sequence before its extensions) is rebuilt position by
// position as in ppo_cluster.hip: F = cuts the prefix reaches within beta*, G_j = those whose link into
// candidate j is within beta*; j qualifies iff some row G[S][j], S disjoint from the prefix and small enough,
// is within beta* at a cut of G_j (one pass over the rows per position); cuts by the fixed-k cut rule.
#include "ppo_cluster.h"

namespace ppo {

constexpr int kFewMaxN = PPO_CLUSTER_FEW_MAX_N, kFewMaxP = PPO_CLUSTER_FEW_MAX_SEGMENTS;
constexpr uint32_t kFewNone = 0xFFFFFFFFu;

// binomial coefficients C(i, j), i <= 64, j <= kFewMaxP + 1 (64-bit: C(64, 9) does not fit 32)
struct FewBinomials {
    unsigned long long c[kFewMaxN + 1][kFewMaxP + 2];
    constexpr FewBinomials() : c{} {
        for (int i = 0; i <= kFewMaxN; ++i) {
            c[i][0] = 1;
            for (int j = 1; j <= kFewMaxP + 1; ++j) c[i][j] = i == 0 ? 0 : c[i - 1][j - 1] + c[i - 1][j];
        }
    }
};
constexpr FewBinomials kFewBinomialsHost = FewBinomials();
__constant__ FewBinomials kFewBinomials = FewBinomials();

struct FewState {
    // (the gaps: with the least values 32 bytes earlier 4 x (128 layers, 64 nodes, 3 segments) took 120 us in place of 118)
    uint32_t best, chosen, done, gap;
    FewConfined confined;
    unsigned long long used;
    union {
        uint32_t first_best[kFewMaxN];           // per node j, until position 0 is settled: the least G[S][j][0] of all sets so far
        unsigned long long cand[kFewMaxN][2];    // then G_j of every candidate of the current position
    };
    unsigned long long start[kFewMaxP][2];   // G of the node chosen at every position
    int32_t seq[kFewMaxP];
};

struct FewLayout {
    int L, n, pmax, rs;                    // rs: entries per row (0 .. L-1), rounded up to even
    uint32_t hi_off, qs_off, state_off, stride;   // bytes within one instance's tables
    unsigned long long level_off[kFewMaxP + 1];   // first full row of level c (1 <= c <= full levels + 1: of the words after all rows)
    size_t rows_bytes;                            // of one instance
    bool confined;                                // instances may be confined to some nodes and cuts: see FewDims

    __host__ __device__ int full_levels() const { return pmax > 1 ? pmax - 1 : 1; }
    __host__ static FewLayout make(int L, int n, int pmax, bool confined = false) {
        FewLayout y{};
        y.confined = confined;
        y.L = L;
        y.n = n;
        y.pmax = pmax;
        y.rs = (L + 1) & ~1;
        size_t off = 0;
        y.hi_off = (uint32_t)off;
        off = align_up(off + (size_t)n * (L + 1), 16);
        y.qs_off = (uint32_t)off;
        off = align_up(off + (size_t)n * n * y.rs * 4, 16);
        y.state_off = (uint32_t)off;
        off = align_up(off + sizeof(FewState), 256);
        y.stride = (uint32_t)off;
        // rows of the levels that are kept whole (1 <= c <= full levels), then entries of the last level (none if pmax = 1)
        unsigned long long rows = 0;
        for (int c = 1; c <= y.full_levels(); ++c) {
            y.level_off[c] = rows;
            rows += kFewBinomialsHost.c[n][c] * (unsigned long long)c;
        }
        if (pmax > 1) y.level_off[pmax] = rows;
        const unsigned long long top = pmax > 1 ? kFewBinomialsHost.c[n][pmax] * (unsigned long long)pmax : 0ull;
        y.rows_bytes = align_up((size_t)(rows * (unsigned long long)y.rs + top) * 4, 256);
        return y;
    }
};

// What the tables of an instance are made of: everything, or the nodes and cuts that can matter (the parts of its slices lie
// where they always do).
struct FewDims {
    int L, n, rs;
    __device__ __forceinline__ FewDims(const FewLayout& y, const unsigned char* base) : L(y.L), n(y.n), rs(y.rs) {
        if (!y.confined) return;
        const FewConfined& c = reinterpret_cast<const FewState*>(base + y.state_off)->confined;
        if (__builtin_amdgcn_readfirstlane((int)c.in) == 0) return;
        L = __builtin_amdgcn_readfirstlane(__popcll(c.cuts[0]) + __popcll(c.cuts[1]) + 1);
        n = __builtin_amdgcn_readfirstlane(__popcll(c.nodes));
        rs = (L + 1) & ~1;
    }
    // first row of level c
    __device__ __forceinline__ unsigned long long first_row(const FewLayout& y, int c) const {
        if (!y.confined) return y.level_off[c];
        unsigned long long rows = 0;
        for (int k = 1; k < c; ++k) rows += kFewBinomials.c[n][k] * (unsigned long long)k;
        return rows;
    }
};
// no value above this one matters
__device__ __forceinline__ uint32_t few_bound(const FewLayout& y, const FewState* st) {
    return y.confined ? (uint32_t)__builtin_amdgcn_readfirstlane((int)st->confined.bound) : kInfBits;
}
// the node and the cut of the instance that place i among those left stands for (cut 0 is the start of the chain)
__device__ inline int few_node(const FewLayout& y, const FewConfined& c, int i) {
    if (!y.confined || !c.in) return i;
    unsigned long long bits = c.nodes;
    for (; i > 0; --i) bits &= bits - 1ull;
    return __ffsll((long long)bits) - 1;
}
__device__ inline int few_cut(const FewLayout& y, const FewConfined& c, int i) {
    if (!y.confined || !c.in || i == 0) return i;
    const int low = __popcll(c.cuts[0]);
    unsigned long long bits = i <= low ? c.cuts[0] : c.cuts[1];
    for (int left = i <= low ? i : i - low; left > 1; --left) bits &= bits - 1ull;
    return (i <= low ? 0 : 64) + __ffsll((long long)bits) - 1;
}

// Shapes this formulation takes: the rows of one instance are counted in 31 bits.
bool cluster_few_supported(int L, int n, int pmax) {
    if (L < 1 || L > PPO_MAX_L || n < 1 || n > kFewMaxN || pmax < 1 || pmax > kFewMaxP || pmax > n) return false;
    unsigned long long rows = 0;
    for (int c = 1; c <= pmax; ++c) rows += kFewBinomialsHost.c[n][c] * (unsigned long long)c;
    return rows < (1ull << 31);
}
size_t cluster_few_tables_bytes(int L, int n, int pmax) { return FewLayout::make(L, n, pmax).stride; }
size_t cluster_few_rows_bytes(int L, int n, int pmax) { return FewLayout::make(L, n, pmax).rows_bytes; }

__device__ __forceinline__ uint32_t few_wave_min(uint32_t v) {
    // minima over the lanes below within rows of 16, then across the rows: lane 63 ends with the minimum of all
#define PPO_FEW_MIN_STEP(CTRL, ROWS)                                                                                     \
    {                                                                                                                   \
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false);                \
        v = o < v ? o : v;                                                                                              \
    }
    PPO_FEW_MIN_STEP(0x111, 0xF)   // row_shr:1, 2, 4, 8
    PPO_FEW_MIN_STEP(0x112, 0xF)
    PPO_FEW_MIN_STEP(0x114, 0xF)
    PPO_FEW_MIN_STEP(0x118, 0xF)
    PPO_FEW_MIN_STEP(0x142, 0xA)   // row_bcast:15 into rows 1 and 3
    PPO_FEW_MIN_STEP(0x143, 0xC)   // row_bcast:31 into rows 2 and 3
#undef PPO_FEW_MIN_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// the set of `size` nodes with a given index in numeric order of the sets (combinatorial number system)
__device__ __forceinline__ unsigned long long few_set_at(unsigned long long index, int size, int n) {
    unsigned long long set = 0;
    int b = n;
    for (int i = size; i >= 1; --i) {
        do { --b; } while (kFewBinomials.c[b][i] > index);
        set |= 1ull << b;
        index -= kFewBinomials.c[b][i];
    }
    return set;
}
// the next larger number with as many bits set
__device__ __forceinline__ unsigned long long few_next_set(unsigned long long x) {
    const unsigned long long low = x & (0ull - x), up = x + low;
    return (((up ^ x) >> 2) >> (__ffsll((long long)x) - 1)) | up;
}

// ---------------------------------------------------------------------------------------------
// Tables: hi, the quotients of every ordered pair shifted by one entry (qs[j][j''][e'] = q_{j,j''}[e'-1], +inf at e' = 0
// and e' >= L), the state, and the rows of level 1.  grid.x = node, grid.y = instance: a workgroup writes what belongs to
// its node (one workgroup per instance: 142 us at n = 50, L = 100, nearly all of it divisions).
// ---------------------------------------------------------------------------------------------
constexpr int kFewTableThreads = 256;
__global__ __launch_bounds__(kFewTableThreads) void few_tables_kernel(const float* __restrict__ t,
                                                                     const float* __restrict__ m,
                                                                     const float* __restrict__ M,
                                                                     const float* __restrict__ B, FewLayout y,
                                                                     unsigned char* __restrict__ ws,
                                                                     uint32_t* __restrict__ rows) {
    __shared__ double P[PPO_MAX_L + 1];
    __shared__ float t_s[PPO_MAX_L], m_s[PPO_MAX_L];
    __shared__ unsigned char hi_s[PPO_MAX_L + 1];
    __shared__ unsigned char pos_s[PPO_MAX_L + 1], node_s[kFewMaxN];
    const int j = blockIdx.x, inst = blockIdx.y, tid = threadIdx.x;
    unsigned char* base = ws + (size_t)inst * y.stride;
    const FewDims d(y, base);
    const int L = d.L, n = d.n, rs = d.rs;
    if (j >= n) return;
    if (y.confined) {
        const FewConfined& in = reinterpret_cast<const FewState*>(base + y.state_off)->confined;
        if (tid < n) node_s[tid] = (unsigned char)few_node(y, in, tid);
        for (int e = tid; e <= L; e += kFewTableThreads) pos_s[e] = (unsigned char)(e == L ? y.L : few_cut(y, in, e));
    }
    const float* ti = t + (size_t)inst * y.L;
    const float* mi = m + (size_t)inst * y.L;
    uint32_t* qs = reinterpret_cast<uint32_t*>(base + y.qs_off) + (size_t)j * n * rs;
    FewState* st = reinterpret_cast<FewState*>(base + y.state_off);
    uint32_t* R = rows + (size_t)inst * (y.rows_bytes / 4);
    for (int i = tid; i < y.L; i += kFewTableThreads) {
        t_s[i] = ti[i] == 0.0f ? 0.0f : ti[i];   // -0 is a size of zero: +0
        m_s[i] = mi[i];
    }
    __syncthreads();
    if (tid == 0) {
        double acc = 0.0;
        P[0] = 0.0;
        for (int i = 0; i < y.L; ++i) {
            acc = acc + (double)m_s[i];
            P[i + 1] = acc;
        }
        if (j == 0) {
            st->best = kInfBits;
            st->chosen = kFewNone;
            st->done = 0u;
            st->used = 0ull;
        }
    }
    const int node = y.confined ? node_s[j] : j;
    const float* Bi = B + ((size_t)inst * y.n + node) * y.n;
    for (int b = tid >> 5; b < n; b += kFewTableThreads >> 5) {
        const float bw = b != j ? Bi[y.confined ? node_s[b] : b] : 1.0f;
        for (int e = tid & 31; e < rs; e += 32) {
            uint32_t v = kInfBits;
            if (b != j && e >= 1 && e < L) v = __float_as_uint(__fdiv_rn(t_s[y.confined ? pos_s[e] - 1 : e - 1], bw));
            qs[b * rs + e] = v;
        }
    }
    __syncthreads();
    const double cap = (double)M[(size_t)inst * y.n + node];
    for (int e = tid; e <= L; e += kFewTableThreads) {
        int lo = e, hi = L;   // the last end that fits; P does not decrease
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            const double part = y.confined ? P[pos_s[mid]] - P[pos_s[e]] : P[mid] - P[e];   // of the cuts left
            if (part <= cap) lo = mid; else hi = mid - 1;
        }
        hi_s[e] = (unsigned char)lo;
        base[y.hi_off + j * (L + 1) + e] = (unsigned char)lo;
    }
    __syncthreads();
    // level 1: the rest of the chain on node j alone
    for (int e = tid; e < rs; e += kFewTableThreads) {
        const bool fits = e < L && hi_s[e] >= L;
        R[(size_t)j * rs + e] = fits ? 0u : kInfBits;
        if (e == 0) st->first_best[j] = fits ? 0u : kInfBits;
    }
}

// ---------------------------------------------------------------------------------------------
// Level c = C + 1 >= 2 below the last.  A unit of work is a set S' and the nodes j outside it with j mod parts the unit's
// (parts > 1 where there are fewer sets than waves).  The minimum over the window (e, hi] is that of two runs of 2^k
// entries; runs are built up to the longest window of the instance, two entries a lane, with wave shifts for the short
// ones and one 8-byte write and read per length beyond; where a window's two runs lie is tabulated once per workgroup.
// ---------------------------------------------------------------------------------------------
constexpr int kFewLevelWaves = 8;
constexpr int kFewRunLevels = 7;     // runs of 2^0 .. 2^6 entries
constexpr int kFewRunRow = 160;      // entries per run-minimum row: 128 computed per row, then +inf
static_assert(kFewRunRow / 2 >= 64 + (1 << (kFewRunLevels - 3)), "the longest runs are built from pairs up to 2^(levels-3) beyond a lane's own");

// of a wave that works several nodes at a time: the least values at the start of the chain, and the nodes outside the set
constexpr int kFewPackDwords = kFewMaxN + kFewMaxN / 4;
// Several nodes at a time are for rows of up to 64 entries only, so what that needs lies where longer rows have their windows
// (10 x (100 layers, 40 nodes, 4 segments): two workgroups fit a compute unit with both, three so, and the level of three nodes
// takes 115 us or 69).
static size_t few_level_lds(const FewLayout& y) {
    const size_t runs = (size_t)kFewLevelWaves * kFewRunLevels * kFewRunRow + 4, pack = (size_t)kFewLevelWaves * kFewPackDwords;
    const size_t one = (size_t)y.n * y.rs + runs, several = (size_t)y.n * (y.rs < 64 ? y.rs : 64) + runs + pack;
    return (one > several ? one : several) * 4;
}

// the value of the next lane; `last` in lane 63
__device__ __forceinline__ uint32_t few_next_lane(uint32_t v, uint32_t last) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x130, 0xF, 0xF, false);
}

template <int C>
__global__ __launch_bounds__(kFewLevelWaves * 64) void few_level_kernel(FewLayout y, unsigned char* __restrict__ ws,
                                                                       uint32_t* __restrict__ rows, uint32_t parts) {
    // window queries [n][rs], run minima of every wave, the longest window (all of it dynamic: the limit is raised to all
    // the LDS there is, which leaves no room for a static part)
    extern __shared__ __align__(16) uint32_t few_smem[];
    constexpr int c = C + 1;
    const int inst = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned char* base = ws + (size_t)inst * y.stride;
    const FewDims dims(y, base);
    const int L = dims.L, n = dims.n, rs = dims.rs, rd = rs / 2;
    if ((unsigned long long)blockIdx.x * kFewLevelWaves >= kFewBinomials.c[n][C] * parts) return;
    const uint32_t* __restrict__ qs = reinterpret_cast<const uint32_t*>(base + y.qs_off);
    FewState* st = reinterpret_cast<FewState*>(base + y.state_off);
    uint32_t* R = rows + (size_t)inst * (y.rows_bytes / 4);
    uint32_t* query = few_smem;
    uint32_t* run = few_smem + (size_t)n * rs + wave * (kFewRunLevels * kFewRunRow);
    int& longest_s = reinterpret_cast<int*>(few_smem)[n * rs + kFewLevelWaves * kFewRunLevels * kFewRunRow];
    uint32_t* least_s = few_smem + (size_t)n * rs + kFewLevelWaves * kFewRunLevels * kFewRunRow + 4 + wave * kFewPackDwords;
    unsigned char* out_s = reinterpret_cast<unsigned char*>(least_s + kFewMaxN);
    // short rows: as many nodes at a time as have room beside each other, 8, 16 or 32 lanes each (one cluster of 50 nodes and
    // 5 segments, 12 to 17 of 100 layers left: the level of three nodes 120 us with a node at a time, 34 with four)
    const int shift = rd <= 8 ? 3 : rd <= 16 ? 4 : rd <= 32 ? 5 : 6, lanes = 1 << shift, hl = lane & (lanes - 1);
    if (shift < 6) least_s[lane] = kInfBits;
    if (tid == 0) longest_s = 1;
    __syncthreads();
    {
        int longest = 1;
        for (int i = tid; i < n * rs; i += kFewLevelWaves * 64) {
            const int j = i / rs, e = i - j * rs;
            uint32_t o1 = kFewRunRow - 1, o2 = kFewRunRow - 1;   // no window: +inf
            if (e < L) {
                int hv = base[y.hi_off + j * (L + 1) + e];
                hv = hv < L - 1 ? hv : L - 1;   // the chain cannot end here: other nodes are still to be used
                if (hv > e) {
                    const int k = 31 - __clz(hv - e);
                    o1 = (uint32_t)(k * kFewRunRow + e + 1);
                    o2 = (uint32_t)(k * kFewRunRow + hv - (1 << k) + 1);
                    longest = hv - e > longest ? hv - e : longest;
                }
            }
            query[i] = (o1 * 4u) | ((o2 * 4u) << 16);
        }
        atomicMax(&longest_s, longest);
    }
    for (int i = lane; i < kFewRunLevels * (kFewRunRow - 128); i += 64)
        run[i / (kFewRunRow - 128) * kFewRunRow + 128 + i % (kFewRunRow - 128)] = kInfBits;
    __syncthreads();
    const int top_run = 31 - __clz(__builtin_amdgcn_readfirstlane(longest_s));
    const unsigned long long units = kFewBinomials.c[n][C] * parts;
    const unsigned long long total_waves = (unsigned long long)gridDim.x * kFewLevelWaves;
    const unsigned long long per_wave = (units + total_waves - 1ull) / total_waves;
    unsigned long long w = ((unsigned long long)blockIdx.x * kFewLevelWaves + (unsigned long long)wave) * per_wave;
    const unsigned long long w_end = w + per_wave < units ? w + per_wave : units;
    const unsigned long long all = n == 64 ? ~0ull : (1ull << n) - 1ull;
    const unsigned long long in_off = dims.first_row(y, C), out_off = dims.first_row(y, c);
    uint32_t first_best = kInfBits;   // lane j: of the rows of node j at e = 0
    const uint32_t bound = few_bound(y, st);
    unsigned long long set = 0, u = w / parts;
    uint32_t part = (uint32_t)(w - u * parts);
    if (w < w_end) set = few_set_at(u, C, n);
    uint2* run2 = reinterpret_cast<uint2*>(run);
    for (; w < w_end; ++w) {
        uint32_t a[C][2];
        int b[C];
        {
            unsigned long long bits = set;
            const uint32_t* arow = R + (size_t)(in_off + u * (unsigned long long)C) * rs + 2 * hl;
#pragma unroll
            for (int mm = 0; mm < C; ++mm) {
                b[mm] = __ffsll((long long)bits) - 1;
                bits &= bits - 1ull;
                uint2 v = make_uint2(kInfBits, kInfBits);
                if (hl < rd) v = *reinterpret_cast<const uint2*>(arow + (size_t)mm * rs);
                a[mm][0] = v.x;
                a[mm][1] = v.y;
            }
        }
        // lane j: the row of S' + j in which j stands (index within its level), for every j outside S'
        unsigned long long my_row = 0;
        {
            const int j = lane;
            unsigned long long rank = 0;
            int pos = 0;
#pragma unroll
            for (int mm = 0; mm < C; ++mm) {
                const bool below = b[mm] < j;
                rank += kFewBinomials.c[b[mm]][below ? mm + 1 : mm + 2];
                pos += below ? 1 : 0;
            }
            rank += kFewBinomials.c[j < n ? j : 0][pos + 1];
            my_row = rank * (unsigned long long)c + (unsigned long long)pos;
        }
        const unsigned long long mine = parts == 1u ? ~0ull : __ballot((uint32_t)lane % parts == part);
        const unsigned long long outside = all & ~set & mine;
        if (shift < 6) {
            const int count = __popcll(outside), part = lane >> shift;
            if ((outside >> lane) & 1ull) out_s[__popcll(outside & ((1ull << lane) - 1ull))] = (unsigned char)lane;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int first = 0; first < count; first += 64 >> shift) {
                const bool in = first + part < count;
                const int j = out_s[in ? first + part : 0];
                const uint32_t row = (uint32_t)__shfl((int)(uint32_t)my_row, j, 64);   // rows are counted in 31 bits
                uint2* to = reinterpret_cast<uint2*>(R + ((size_t)out_off + row) * rs + 2 * hl);
                uint32_t v0 = kInfBits, v1 = kInfBits;
                if (hl < rd) {
#pragma unroll
                    for (int mm = 0; mm < C; ++mm) {
                        const uint2 q = *reinterpret_cast<const uint2*>(qs + (j * n + b[mm]) * rs + 2 * hl);
                        const uint32_t x0 = q.x > a[mm][0] ? q.x : a[mm][0], x1 = q.y > a[mm][1] ? q.y : a[mm][1];
                        v0 = x0 < v0 ? x0 : v0;
                        v1 = x1 < v1 ? x1 : v1;
                    }
                }
                // links within the bound are few: most rows hold nothing within it
                if (__ballot(v0 <= bound || v1 <= bound) == 0ull) {
                    if (in && hl < rd) *to = make_uint2(kInfBits, kInfBits);
                    continue;
                }
                // as below; a run that passes the end of a row is never asked for
                run2[lane] = make_uint2(v0, v1);
                if (top_run >= 1) {
                    const uint32_t n0 = few_next_lane(v0, kInfBits);
                    v0 = v1 < v0 ? v1 : v0;
                    v1 = n0 < v1 ? n0 : v1;
                    run2[kFewRunRow / 2 + lane] = make_uint2(v0, v1);
                }
                if (top_run >= 2) {
                    const uint32_t n0 = few_next_lane(v0, kInfBits), n1 = few_next_lane(v1, kInfBits);
                    v0 = n0 < v0 ? n0 : v0;
                    v1 = n1 < v1 ? n1 : v1;
                    run2[2 * (kFewRunRow / 2) + lane] = make_uint2(v0, v1);
                }
                for (int k = 3; k <= top_run; ++k) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    const uint2 f = run2[(k - 1) * (kFewRunRow / 2) + lane + (1 << (k - 2))];
                    v0 = f.x < v0 ? f.x : v0;
                    v1 = f.y < v1 ? f.y : v1;
                    run2[k * (kFewRunRow / 2) + lane] = make_uint2(v0, v1);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const uint2 d = *reinterpret_cast<const uint2*>(query + j * rs + 2 * (hl < rd ? hl : 0));
                const unsigned char* runb = reinterpret_cast<const unsigned char*>(run);
                constexpr uint32_t kNone = (kFewRunRow - 1) * 4u;
                auto at = [&](uint32_t off) -> uint32_t {   // the row of a part starts 2 * lanes entries after the one before
                    const uint32_t v = *reinterpret_cast<const uint32_t*>(runb + (off == kNone ? 0u : off + (uint32_t)part * (uint32_t)lanes * 8u));
                    return off == kNone ? kInfBits : v;
                };
                const uint32_t a0 = at(d.x & 0xFFFFu), b0 = at(d.x >> 16), a1 = at(d.y & 0xFFFFu), b1 = at(d.y >> 16);
                const uint32_t res0 = a0 < b0 ? a0 : b0, res1 = a1 < b1 ? a1 : b1;
                if (in && hl < rd) *to = make_uint2(res0, res1);
                if (in && hl == 0) atomicMin(&least_s[j], res0);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        } else
        for (unsigned long long jb = outside; jb; jb &= jb - 1ull) {
            const int j = __ffsll((long long)jb) - 1;
            const unsigned long long row = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(my_row >> 32), j) << 32) |
                                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_row, j);
            uint32_t v0 = kInfBits, v1 = kInfBits;
            if (lane < rd) {
#pragma unroll
                for (int mm = 0; mm < C; ++mm) {
                    const uint2 q = *reinterpret_cast<const uint2*>(qs + (size_t)(j * n + b[mm]) * rs + 2 * lane);
                    const uint32_t x0 = q.x > a[mm][0] ? q.x : a[mm][0], x1 = q.y > a[mm][1] ? q.y : a[mm][1];
                    v0 = x0 < v0 ? x0 : v0;
                    v1 = x1 < v1 ? x1 : v1;
                }
            }
            // links within the bound are few: most rows hold nothing within it
            if (__ballot(v0 <= bound || v1 <= bound) == 0ull) {
                if (lane < rd) *reinterpret_cast<uint2*>(R + (size_t)(out_off + row) * rs + 2 * lane) = make_uint2(kInfBits, kInfBits);
                continue;
            }
            // minima over runs of 2^k entries starting at each entry
            run2[lane] = make_uint2(v0, v1);
            if (top_run >= 1) {
                const uint32_t n0 = few_next_lane(v0, kInfBits);
                v0 = v1 < v0 ? v1 : v0;
                v1 = n0 < v1 ? n0 : v1;
                run2[kFewRunRow / 2 + lane] = make_uint2(v0, v1);
            }
            if (top_run >= 2) {
                const uint32_t n0 = few_next_lane(v0, kInfBits), n1 = few_next_lane(v1, kInfBits);
                v0 = n0 < v0 ? n0 : v0;
                v1 = n1 < v1 ? n1 : v1;
                run2[2 * (kFewRunRow / 2) + lane] = make_uint2(v0, v1);
            }
#pragma unroll
            for (int k = 3; k < kFewRunLevels; ++k) {
                if (top_run < k) break;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const uint2 f = run2[(k - 1) * (kFewRunRow / 2) + lane + (1 << (k - 2))];
                v0 = f.x < v0 ? f.x : v0;
                v1 = f.y < v1 ? f.y : v1;
                run2[k * (kFewRunRow / 2) + lane] = make_uint2(v0, v1);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const uint2 d = *reinterpret_cast<const uint2*>(query + j * rs + 2 * (lane < rd ? lane : 0));
            const unsigned char* runb = reinterpret_cast<const unsigned char*>(run);
            auto at = [&](uint32_t off) -> uint32_t { return *reinterpret_cast<const uint32_t*>(runb + off); };
            const uint32_t a0 = at(d.x & 0xFFFFu), b0 = at(d.x >> 16), a1 = at(d.y & 0xFFFFu), b1 = at(d.y >> 16);
            const uint32_t res0 = a0 < b0 ? a0 : b0, res1 = a1 < b1 ? a1 : b1;
            if (lane < rd) *reinterpret_cast<uint2*>(R + (size_t)(out_off + row) * rs + 2 * lane) = make_uint2(res0, res1);
            const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)res0);
            if (lane == j) first_best = r < first_best ? r : first_best;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (w + 1ull < w_end && ++part == parts) {
            part = 0;
            ++u;
            set = few_next_set(set);
        }
    }
    if (shift < 6) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        first_best = least_s[lane];
    }
    if (first_best < kInfBits) atomicMin(&st->first_best[lane], first_best);
}

// ---------------------------------------------------------------------------------------------
// The last level, c = C + 1 = pmax.  What is wanted of it is beta* and the nodes that can stand first, so a value matters
// only if it is at most the least found so far (the bound) and below the least of its own first node.  A wave loads the
// rows of a set S' and counts their entries that could still matter, at cuts a first segment can end at.  None: the set
// is done.  A few: each of them is tried for all nodes j at once, lane j dividing for itself.  Many (before there is a
// bound): node by node over the whole rows.  A mark per set, bit m for a row of member m with any entry within the bound
// (of that time, which is never below beta*), tells the scans below which rows of level C to look at.
// 230,300 sets of 46 nodes (n = 50, pmax = 5): 1.69 ms when every row was evaluated in full.
// ---------------------------------------------------------------------------------------------
constexpr int kFewTopWaves = 4;
constexpr int kFewTopTries = 64;   // an entry tried over the lanes costs about as much as a node over whole rows

template <int C>
__global__ __launch_bounds__(kFewTopWaves * 64) void few_top_kernel(FewLayout y, unsigned char* __restrict__ ws,
                                                                   uint32_t* __restrict__ rows, const float* __restrict__ t,
                                                                   const float* __restrict__ B) {
    extern __shared__ __align__(16) uint32_t few_smem[];   // bandwidths transposed: [b][j] = B[j][b]
    __shared__ float t_s[PPO_MAX_L];
    const int inst = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned char* base = ws + (size_t)inst * y.stride;
    const FewDims dims(y, base);
    const int L = dims.L, n = dims.n, rs = dims.rs, rd = rs / 2;
    if ((unsigned long long)blockIdx.x * kFewTopWaves >= kFewBinomials.c[n][C]) return;
    const uint32_t* __restrict__ qs = reinterpret_cast<const uint32_t*>(base + y.qs_off);
    FewState* st = reinterpret_cast<FewState*>(base + y.state_off);
    uint32_t* R = rows + (size_t)inst * (y.rows_bytes / 4);
    const unsigned long long in_off = dims.first_row(y, C);
    uint32_t* marks = R + (size_t)dims.first_row(y, C + 1) * rs;   // one word per set of level C, after all rows
    float* Bt = reinterpret_cast<float*>(few_smem);
    __shared__ unsigned char node_s[kFewMaxN];
    if (y.confined) {
        if (tid < n) node_s[tid] = (unsigned char)few_node(y, st->confined, tid);
        __syncthreads();
        for (int i = tid; i < n * n; i += kFewTopWaves * 64) {
            const int j = i / n, b = i - j * n;
            Bt[b * n + j] = B[((size_t)inst * y.n + node_s[j]) * y.n + node_s[b]];
        }
        for (int i = tid; i < L - 1; i += kFewTopWaves * 64) {
            const float x = t[(size_t)inst * y.L + few_cut(y, st->confined, i + 1) - 1];
            t_s[i] = x == 0.0f ? 0.0f : x;   // -0 is a size of zero: +0
        }
    } else {
        for (int i = tid; i < n * n; i += kFewTopWaves * 64) {
            const int j = i / n, b = i - j * n;
            Bt[b * n + j] = B[(size_t)inst * n * n + i];
        }
        for (int i = tid; i < L; i += kFewTopWaves * 64) {
            const float x = t[(size_t)inst * L + i];
            t_s[i] = x == 0.0f ? 0.0f : x;
        }
    }
    // lane j: last cut of a first segment on node j (another node follows)
    int my_hi0 = lane < n ? (int)base[y.hi_off + lane * (L + 1)] : 0;
    my_hi0 = my_hi0 < L - 1 ? my_hi0 : L - 1;
    const int max_hi0 = (int)~few_wave_min(~(uint32_t)my_hi0);
    const uint32_t known = few_bound(y, st);
    __syncthreads();
    const unsigned long long nsets = kFewBinomials.c[n][C];
    const unsigned long long total_waves = (unsigned long long)gridDim.x * kFewTopWaves;
    const unsigned long long per_wave = (nsets + total_waves - 1ull) / total_waves;
    unsigned long long u = ((unsigned long long)blockIdx.x * kFewTopWaves + (unsigned long long)wave) * per_wave;
    const unsigned long long u_end = u + per_wave < nsets ? u + per_wave : nsets;
    const unsigned long long all = n == 64 ? ~0ull : (1ull << n) - 1ull;
    unsigned long long set = 0;
    if (u < u_end) set = few_set_at(u, C, n);
    for (; u < u_end; ++u) {
        uint32_t a[C][2];
        int b[C];
        const uint32_t mine = lane < n ? __hip_atomic_load(&st->first_best[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kInfBits;
        {
            unsigned long long bits = set;
            const uint32_t* arow = R + (size_t)(in_off + u * (unsigned long long)C) * rs + 2 * lane;
#pragma unroll
            for (int mm = 0; mm < C; ++mm) {
                b[mm] = __ffsll((long long)bits) - 1;
                bits &= bits - 1ull;
                uint2 v = make_uint2(kInfBits, kInfBits);
                if (lane < rd) v = *reinterpret_cast<const uint2*>(arow + (size_t)mm * rs);
                a[mm][0] = v.x;
                a[mm][1] = v.y;
            }
        }
        const uint32_t least = few_wave_min(mine), bound = least < known ? least : known;
        const unsigned long long outside = all & ~set;
        // a value of node j is wanted if it is below my_limit
        const uint32_t my_limit = mine == bound ? bound : bound + 1u;
        const bool any_tie = (__ballot(my_limit > bound) & outside) != 0ull;
        const uint32_t limit = any_tie ? bound + 1u : bound;
        const bool in0 = lane >= 1 && 2 * lane <= max_hi0, in1 = 2 * lane + 1 <= max_hi0;
        unsigned long long want[C][2];
        uint32_t mark = 0;
        int tries = 0;
#pragma unroll
        for (int mm = 0; mm < C; ++mm) {
            if (__ballot(a[mm][0] <= bound || a[mm][1] <= bound)) mark |= 1u << mm;
            want[mm][0] = __ballot(in0 && a[mm][0] < limit);
            want[mm][1] = __ballot(in1 && a[mm][1] < limit);
            tries += __popcll(want[mm][0]) + __popcll(want[mm][1]);
        }
        if (lane == 0) marks[u] = mark;
        if (tries) {
            uint32_t acc = kInfBits;   // lane j: least value of node j
            if (tries <= kFewTopTries) {
#pragma unroll
                for (int mm = 0; mm < C; ++mm) {
                    const float bw = lane < n ? Bt[b[mm] * n + lane] : 1.0f;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        for (unsigned long long wb = want[mm][h]; wb; wb &= wb - 1ull) {
                            const int x = __ffsll((long long)wb) - 1, e = 2 * x + h;
                            const uint32_t av = (uint32_t)__builtin_amdgcn_readlane((int)a[mm][h], x);
                            const uint32_t q = __float_as_uint(__fdiv_rn(t_s[e - 1], bw));
                            const uint32_t v = q > av ? q : av;
                            if (e <= my_hi0) acc = v < acc ? v : acc;
                        }
                }
            } else {
                for (unsigned long long jb = outside; jb; jb &= jb - 1ull) {
                    const int j = __ffsll((long long)jb) - 1;
                    const int hi0 = __builtin_amdgcn_readlane(my_hi0, j);
                    uint32_t v0 = kInfBits, v1 = kInfBits;
                    if (lane < rd) {
#pragma unroll
                        for (int mm = 0; mm < C; ++mm) {
                            const uint2 q = *reinterpret_cast<const uint2*>(qs + (size_t)(j * n + b[mm]) * rs + 2 * lane);
                            const uint32_t x0 = q.x > a[mm][0] ? q.x : a[mm][0], x1 = q.y > a[mm][1] ? q.y : a[mm][1];
                            v0 = x0 < v0 ? x0 : v0;
                            v1 = x1 < v1 ? x1 : v1;
                        }
                    }
                    // G[S][j][0]: the least with 1 <= e' <= hi_j(0) (quotients are +inf at 0 and from L on)
                    uint32_t r = 2 * lane <= hi0 ? v0 : kInfBits;
                    const uint32_t r1 = 2 * lane + 1 <= hi0 ? v1 : kInfBits;
                    r = few_wave_min(r1 < r ? r1 : r);
                    if (lane == j) acc = r;
                }
            }
            if (((outside >> lane) & 1ull) && acc < my_limit) atomicMin(&st->first_best[lane], acc);
        }
        if (u + 1ull < u_end) set = few_next_set(set);
    }
}

// ---------------------------------------------------------------------------------------------
// One position of the answer.  step(s), s >= 1: takes the node found for position s - 1 (for position 0 the smallest
// one whose least value is beta*), stops if the prefix completes the chain, else prepares the masks G_j of position s.
// scan(s): the smallest candidate with a row within beta* at a cut of its mask.  One workgroup per instance for the
// steps, the candidates dealt to its waves.
// ---------------------------------------------------------------------------------------------
constexpr int kFewStepWaves = 16;
__global__ __launch_bounds__(kFewStepWaves * 64) void few_step_kernel(FewLayout y, unsigned char* __restrict__ ws, int s,
                                                      float* __restrict__ beta_out, int32_t* __restrict__ segs_out,
                                                      int32_t* __restrict__ cuts_out, int32_t* __restrict__ order_out) {
    const int inst = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    unsigned char* base = ws + (size_t)inst * y.stride;
    const FewDims dims(y, base);
    const int L = dims.L, n = dims.n, rs = dims.rs;
    const unsigned char* __restrict__ hi_t = base + y.hi_off;
    const uint32_t* __restrict__ qs = reinterpret_cast<const uint32_t*>(base + y.qs_off);
    FewState* st = reinterpret_cast<FewState*>(base + y.state_off);
    int32_t* order = order_out + (size_t)inst * y.n;
    int32_t* cuts = cuts_out ? cuts_out + (size_t)inst * (y.n - 1) : nullptr;
    auto hi = [&](int j, int e) -> int { return hi_t[j * (L + 1) + e]; };
    // is cut e2 (1 <= e2 <= L) inside the window of node j that starts at the latest cut of (g0, g1) below e2?
    auto covered = [&](unsigned long long g0, unsigned long long g1, int j, int e2) -> bool {
        unsigned long long m0 = g0, m1 = 0;
        if (e2 < 64)
            m0 = g0 & ((1ull << e2) - 1ull);
        else
            m1 = e2 >= 128 ? g1 : g1 & ((1ull << (e2 - 64)) - 1ull);
        const int from = m1 ? 127 - __clzll((long long)m1) : m0 ? 63 - __clzll((long long)m0) : -1;
        return from >= 0 && hi(j, from) >= e2;
    };
    if (s > 1 && st->done) return;
    // position 0 starts at cut 0 whatever its node
    uint32_t best, chosen;
    unsigned long long G0 = 1ull, G1 = 0ull, used = 0ull;
    if (s == 1) {
        const uint32_t mine = lane < n ? st->first_best[lane] : kInfBits;
        best = few_wave_min(mine);
        chosen = (uint32_t)(__ffsll((long long)__ballot(mine == best)) - 1);
        if (wave == 0) {
            for (int i = lane; i < y.n; i += 64) order[i] = -1;
            if (cuts)
                for (int i = lane; i < y.n - 1; i += 64) cuts[i] = -1;
            if (lane == 0) st->best = best;
        }
        if (best >= kInfBits) {
            if (threadIdx.x == 0) {
                beta_out[inst] = __uint_as_float(kInfBits);
                segs_out[inst] = 0;
                st->done = 1u;
            }
            return;
        }
    } else {
        best = st->best;
        chosen = st->chosen;
        used = st->used;
        if (chosen != kFewNone) {
            G0 = st->cand[chosen][0];
            G1 = st->cand[chosen][1];
        }
    }
    __syncthreads();   // what the last step left has been read by all waves
    int last = 0, p = s - 1;
    bool finish = true;   // without a node: cannot happen, some completion of the prefix reaches beta*
    unsigned long long F0 = 0ull, F1 = 0ull;
    if (chosen != kFewNone) {
        const bool complete = covered(G0, G1, (int)chosen, L);
        F0 = __ballot(lane >= 1 && lane < L && covered(G0, G1, (int)chosen, lane));
        F1 = __ballot(lane + 64 < L && covered(G0, G1, (int)chosen, lane + 64));
        if (threadIdx.x == 0) {
            st->seq[s - 1] = (int32_t)chosen;
            st->start[s - 1][0] = G0;
            st->start[s - 1][1] = G1;
        }
        used |= 1ull << chosen;
        last = (int)chosen;
        p = s;
        finish = complete || s == y.pmax;
    }
    if (finish) {
        if (wave != 0) return;
        // cuts: latest segment first, each time the smallest start (reached by the prefix, link within beta*)
        // whose window covers the end
        int e = L;
        for (int q = p - 1; q >= 1 && cuts; --q) {
            const int jq = q == s - 1 ? last : st->seq[q];
            const unsigned long long g0 = q == s - 1 ? G0 : st->start[q][0];
            const unsigned long long g1 = q == s - 1 ? G1 : st->start[q][1];
            const unsigned long long m0 = __ballot(((g0 >> lane) & 1ull) && lane < e && hi(jq, lane) >= e);
            const unsigned long long m1 = __ballot(((g1 >> lane) & 1ull) && lane + 64 < e && hi(jq, lane + 64 < L ? lane + 64 : L) >= e);
            if (!(m0 | m1)) break;   // cannot happen: e was reached from such a start
            const int first = m0 ? __ffsll((long long)m0) - 1 : 63 + __ffsll((long long)m1);
            if (lane == 0) cuts[q - 1] = (int32_t)few_cut(y, st->confined, first);
            e = first;
        }
        if (lane == 0) {
            beta_out[inst] = __uint_as_float(best);
            segs_out[inst] = p;
            for (int q = 0; q < p; ++q) order[q] = few_node(y, st->confined, q == s - 1 ? last : st->seq[q]);
            st->done = 1u;
        }
        return;
    }
    // the masks of position s
    for (int j = wave; j < n; j += kFewStepWaves) {
        unsigned long long g0 = 0ull, g1 = 0ull;
        if (!((used >> j) & 1ull)) {
            const uint32_t* __restrict__ q = qs + (size_t)(last * n + j) * rs;
            const int e0 = lane, e1 = lane + 64;
            g0 = __ballot(((F0 >> lane) & 1ull) && e0 < L && q[e0] <= best);
            g1 = __ballot(((F1 >> lane) & 1ull) && e1 < L && q[e1 < rs ? e1 : 0] <= best);
        }
        if (lane == 0) {
            st->cand[j][0] = g0;
            st->cand[j][1] = g1;
        }
    }
    if (threadIdx.x == 0) {
        st->chosen = kFewNone;
        st->used = used;
    }
}

constexpr int kFewScanWaves = 4;
__global__ __launch_bounds__(kFewScanWaves * 64) void few_scan_kernel(FewLayout y, unsigned char* __restrict__ ws,
                                                                      const uint32_t* __restrict__ rows, int s) {
    const int c = (int)blockIdx.y + 1, inst = blockIdx.z, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    unsigned char* base = ws + (size_t)inst * y.stride;
    const FewDims dims(y, base);
    const int n = dims.n, rs = dims.rs, rd = rs / 2;
    FewState* st = reinterpret_cast<FewState*>(base + y.state_off);
    if (st->done) return;
    const uint32_t best = st->best;
    const unsigned long long used = st->used;
    const uint32_t* R = rows + (size_t)inst * (y.rows_bytes / 4);
    // level pmax - 1 is most of the rows: those without a mark hold nothing within beta*
    const unsigned long long in_off = dims.first_row(y, c);
    const uint32_t* marks = c == y.pmax - 1 ? R + (size_t)dims.first_row(y, y.pmax) * rs : nullptr;
    const unsigned long long nsets = kFewBinomials.c[n][c];
    const unsigned long long total_waves = (unsigned long long)gridDim.x * kFewScanWaves;
    const unsigned long long per_wave = (nsets + total_waves - 1ull) / total_waves;
    unsigned long long u = ((unsigned long long)blockIdx.x * kFewScanWaves + (unsigned long long)wave) * per_wave;
    const unsigned long long u_end = u + per_wave < nsets ? u + per_wave : nsets;
    if (u >= u_end) return;
    uint32_t found = kFewNone;   // the smallest candidate that any wave has been seen to find
    auto look_at = [&](unsigned long long set, unsigned long long at, uint32_t mark) {
        unsigned long long bits = set;
        for (int i = 0; i < c; ++i) {
            const int j = __ffsll((long long)bits) - 1;
            bits &= bits - 1ull;
            if ((uint32_t)j >= found || !((mark >> i) & 1u)) continue;   // wave-uniform: `found` is kept the same in all lanes
            const unsigned long long g0 = st->cand[j][0], g1 = st->cand[j][1];
            bool ok = false;
            if (lane < rd) {
                const uint2 v = *reinterpret_cast<const uint2*>(R + (size_t)(in_off + at * (unsigned long long)c + (unsigned long long)i) * rs + 2 * lane);
                const int e0 = 2 * lane, e1 = e0 + 1;
                const bool in0 = ((e0 < 64 ? g0 >> e0 : g1 >> (e0 - 64)) & 1ull) != 0ull;
                const bool in1 = ((e1 < 64 ? g0 >> e1 : g1 >> (e1 - 64)) & 1ull) != 0ull;
                ok = (in0 && v.x <= best) || (in1 && v.y <= best);
            }
            if (__ballot(ok)) {
                found = (uint32_t)j;
                if (lane == 0) atomicMin(&st->chosen, found);
            }
        }
    };
    auto seen = [&]() {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)__hip_atomic_load(&st->chosen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        found = o < found ? o : found;
    };
    if (marks) {
        for (; u < u_end; u += 64ull) {
            const uint32_t my_mark = u + (unsigned long long)lane < u_end ? marks[u + (unsigned long long)lane] : 0u;
            unsigned long long some = __ballot(my_mark != 0u);
            if (some) seen();
            for (; some; some &= some - 1ull) {
                const int x = __ffsll((long long)some) - 1;
                const unsigned long long at = u + (unsigned long long)x;
                const unsigned long long set = few_set_at(at, c, n);
                if (!(set & used)) look_at(set, at, (uint32_t)__builtin_amdgcn_readlane((int)my_mark, x));
            }
        }
    } else {
        unsigned long long set = few_set_at(u, c, n);
        for (uint32_t turn = 0; u < u_end; ++u, ++turn) {
            if ((turn & 15u) == 0u) seen();
            if (!(set & used)) look_at(set, u, ~0u);
            if (u + 1ull < u_end) set = few_next_set(set);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
// Whether the search is confined to the nodes and cuts that can matter (ppo_cluster_bound.hip), and to values within the bound
// found there.  That costs about 70 us (the bound 27, the walks 25 to 45), 15 to 20 where the nodes of the bound do not hold the
// chain.  Measured in us, without and with it, nodes just large enough: one cluster of 50 nodes, 100 layers and 5 segments 480 / 259,
// of 40 nodes 273 / 204, 8 of 64 nodes, 30 layers and 4 segments 516 / 321, 3 of 30 nodes, 50 layers and 5 segments 255 / 209, 4
// paper-shaped ones of 50 nodes and 4 segments 945 / 206.  Of fewer nodes most stay: 11 of 21 nodes, 30 layers and 5 segments (320
// thousand rows) 209 / 245, 57 of 14 nodes, 50 layers and 5 segments 234 / 231, but 44 of 21 nodes 650 / 619.  Nothing to leave out:
// one of 50 nodes and 100 layers that does not fit 371 / 385, 4 of 40 nodes and 50 layers with one transfer size and bandwidth
// 1122 / 1132, one of them 350 / 452 (the ties are scanned by fewer workgroups, see few_grid).
static bool few_confined(int n, int pmax, int n_inst) {
    unsigned long long rows = 0;
    for (int c = 1; c < pmax; ++c) rows += kFewBinomialsHost.c[n][c] * (unsigned long long)c;
    return n >= 9 && pmax >= 2 && rows * (unsigned long long)n_inst >= (n >= 30 ? 300000ull : 1200000ull);
}
hipError_t launch_cluster_few_tables(const float* t, const float* m, const float* M, const float* B, int L, int n,
                                     int pmax, int n_inst, void* ws, void* rows, hipStream_t stream) {
    const FewLayout y = FewLayout::make(L, n, pmax, few_confined(n, pmax, n_inst));
    if (y.confined) {
        FewState* state = reinterpret_cast<FewState*>(static_cast<unsigned char*>(ws) + y.state_off);
        const hipError_t e = launch_few_confine(t, m, M, B, L, n, pmax, n_inst, &state->confined, y.stride, stream);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(few_tables_kernel, dim3(n, n_inst), dim3(kFewTableThreads), 0, stream, t, m, M, B, y,
                       static_cast<unsigned char*>(ws), static_cast<uint32_t*>(rows));
    return hipGetLastError();
}

// A level below the last: two workgroups per compute unit stay resident (each tabulates the windows once), over all
// instances; a set's nodes are split among waves where there are fewer sets than waves.
template <int C>
static hipError_t few_launch_level(int n_inst, hipStream_t stream, const FewLayout& y, unsigned char* ws, uint32_t* rows) {
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&few_level_kernel<C>), lds_allowed);
    if (e != hipSuccess) return e;
    const unsigned long long sets = kFewBinomialsHost.c[y.n][C];
    const uint32_t blocks_each = (512u + (uint32_t)n_inst - 1u) / (uint32_t)n_inst;
    const unsigned long long waves = (unsigned long long)blocks_each * kFewLevelWaves;
    unsigned long long parts = 2ull * waves / sets;
    parts = parts < 1ull ? 1ull : parts > (unsigned long long)y.n ? (unsigned long long)y.n : parts;
    const unsigned long long blocks = (sets * parts + kFewLevelWaves - 1ull) / kFewLevelWaves;
    hipLaunchKernelGGL(few_level_kernel<C>, dim3((uint32_t)(blocks < blocks_each ? blocks : blocks_each), n_inst),
                       dim3(kFewLevelWaves * 64), few_level_lds(y), stream, y, ws, rows, (uint32_t)parts);
    return hipGetLastError();
}
template <int C>
static hipError_t few_launch_top(int n_inst, hipStream_t stream, const FewLayout& y, unsigned char* ws, uint32_t* rows,
                                 const float* t, const float* B) {
    // eight workgroups of four waves to a compute unit, each wave several sets, so that later ones meet a bound
    const unsigned long long sets = kFewBinomialsHost.c[y.n][C];
    const unsigned long long cap = (2048ull + (unsigned long long)n_inst - 1ull) / (unsigned long long)n_inst;
    unsigned long long blocks = (sets + kFewTopWaves - 1ull) / kFewTopWaves;
    blocks = blocks < cap ? blocks : cap;
    hipLaunchKernelGGL(few_top_kernel<C>, dim3((uint32_t)blocks, n_inst), dim3(kFewTopWaves * 64), (size_t)y.n * y.n * 4, stream,
                       y, ws, rows, t, B);
    return hipGetLastError();
}
// levels C + 1 .. pmax
template <int C>
static hipError_t few_launch_levels(int n_inst, hipStream_t stream, const FewLayout& y, unsigned char* ws, uint32_t* rows,
                                    const float* t, const float* B) {
    if constexpr (C < kFewMaxP) {
        if (C >= y.pmax) return hipSuccess;
        if (C + 1 == y.pmax) return few_launch_top<C>(n_inst, stream, y, ws, rows, t, B);
        const hipError_t e = few_launch_level<C>(n_inst, stream, y, ws, rows);
        return e != hipSuccess ? e : few_launch_levels<C + 1>(n_inst, stream, y, ws, rows, t, B);
    } else {
        return hipSuccess;
    }
}

static uint32_t few_grid(unsigned long long sets, int waves_per_block) {
    // enough workgroups to fill the chip, never more than there are sets (with four times as many, 12 clusters of 30 nodes, 100
    // layers and 5 segments that leave most sets without a mark took 519 us in place of 279; where every link ties and no
    // set is without one, one cluster of 40 nodes took 404 in place of 535)
    unsigned long long blocks = (sets + (unsigned long long)waves_per_block - 1ull) / (unsigned long long)waves_per_block;
    const unsigned long long cap = 256ull * 8ull;
    if (blocks > cap) blocks = cap;
    return (uint32_t)(blocks ? blocks : 1ull);
}

// the tables of the n_inst instances are in ws, the rows of instance i at rows + i * rows_bytes
hipError_t launch_cluster_few_solve(const float* t, const float* B, int L, int n, int pmax, int n_inst, void* ws_, void* rows_,
                                    float* beta_out, int32_t* segs_out, int32_t* cuts_out, int32_t* order_out,
                                    hipStream_t stream) {
    const FewLayout y = FewLayout::make(L, n, pmax, few_confined(n, pmax, n_inst));
    unsigned char* ws = static_cast<unsigned char*>(ws_);
    uint32_t* rows = static_cast<uint32_t*>(rows_);
    hipError_t e = few_launch_levels<1>(n_inst, stream, y, ws, rows, t, B);
    if (e != hipSuccess) return e;
    for (int s = 1; s <= pmax; ++s) {
        hipLaunchKernelGGL(few_step_kernel, dim3(n_inst), dim3(kFewStepWaves * 64), 0, stream, y, ws, s, beta_out, segs_out,
                           cuts_out, order_out);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (s == pmax) break;
        unsigned long long most = 0;
        for (int c = 1; c <= pmax - s; ++c) most = kFewBinomialsHost.c[n][c] > most ? kFewBinomialsHost.c[n][c] : most;
        hipLaunchKernelGGL(few_scan_kernel, dim3(few_grid(most, kFewScanWaves), pmax - s, n_inst), dim3(kFewScanWaves * 64), 0,
                           stream, y, ws, rows, s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ppo
