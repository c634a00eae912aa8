// The whole search of ppo_solve in one launch: dynamic programming over the sets of nodes not yet used, one
// workgroup per instance, tables, rows, optimum and traceback included.
//
// The bottleneck of Eq. 2 is a maximum over links, so what is still to be paid from a cut on depends only on the
// node j that takes the next segment, the cut e and the set R of nodes not used before it (j in R):
//     A[{j}][j][e] = 0 if layers [e, L) fit node j, else +inf
//     A[R][j][e]   = min over e' in (e, min(hi_j(e), L-1)] of  min over j'' in R' of max(q_{j,j''}[e'-1], A[R'][j''][e'])
// with R' = R \ j and hi_j(e) the last e' such that layers [e, e') fit node j; beta* = min over j of A[All][j][0].
// k 2^(k-1) rows of L entries replace the k! programmes of the enumeration.  The rows are those of the cluster form
// (ppo_cluster.hip) with every node to be used; there a level is a launch over all instances, here it is a barrier.
//
// Values.  The rows hold 16-bit codes that do not decrease with the quotient: kCodeZero for 0, then kCodeZero + 1 +
// ((bits - lo) >> shift) with [lo, hi] the range of the quotients' binary32 patterns and the least shift that fits, and
// kCodeInf beyond.  Minima and maxima commute with a non-decreasing map, so the search gives the code of beta*.  If
// more than one of the quotients has that code, the search is repeated with [lo, hi] the range of those (everything
// below counts as 0, everything above as +inf): a pass divides the range by 30,000, so there are at most three, and
// after the last one "code <= code of beta*" says the same as "value <= beta*".  No quotient is ranked among the others,
// which is what the tables of the enumeration spend most of their time on.
//
// What bounds it: no single unit.  4096 x (96, 8) issues 47 vector, 44 scalar and 14 LDS instructions a row (tables and
// answer included), which fills 0.55 of the vector, 0.52 of the scalar and 0.38 of the LDS units' time; of the time of its
// seven waves on a SIMD 0.61 is spent waiting: for LDS and the rows below, or at the barriers (the prefix sums and the
// answer are one wave's work; the counter does not tell these apart).  1024 x (50, 6): 0.56, 0.28 and 0.24, six waves, 0.66 waiting.
// Rows of up to 64 entries go two sets to a wave, longer ones leave lanes beyond the chain idle.  Up to 8 nodes one launch
// does everything for an instance in one workgroup (no tables in HBM, no launch gaps); the answer is walked by one wave,
// because run by all of them (redundantly, with barriers) it issued more instructions than the rows did (50 layers on 6
// nodes: 65 us for 1024 instances, 43 with one wave).
// Many instances of long chains on six to eight nodes go by the ranges of cuts that a set can meet (ppo_bands.hip).
// Measured on one MI355X, per call with scratch and outputs kept (in brackets with the call's own scratch; the enumeration
// before): 256 x (L 12, k 4) 18 us (21; 58), 1024 x (50, 6) 44 us (43; 163), 37 x (127, 9) 87 us (91; 97 ms), 1 x (64, 11) 76 us
// (92; 3.2 ms).
#include "ppo_sets.h"

namespace ppo {

// ppo_bands.hip
bool bands_apply(int L, int k, int n_inst, size_t slot, size_t slot_count);
hipError_t launch_bands_solve(const float*, const float*, const float*, const float*, int, int, int, float*, int32_t*, int32_t*, void*,
                              size_t, size_t, hipStream_t);

namespace {

constexpr int kRunLevels = 7;                             // minima over runs of 2^0 .. 2^6 entries
// Run rows of a wave: 64 dwords each (rows of 128 entries take runs of up to 2^6 of them, rows of 64 up to 2^5), then
// entries that are +inf, for windows that are empty.
constexpr int run_levels(int G) { return G == 1 ? kRunLevels : kRunLevels - 1; }
constexpr int run_dwords(int G) { return run_levels(G) * 64 + 48; }
constexpr uint32_t no_window(int G) { return (uint32_t)run_levels(G) * 256u; }   // byte offset of the first of those
constexpr uint32_t kFinestCodes = kCodeInf - kCodeZero - 2u;   // buckets of the code

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}
__device__ __forceinline__ uint32_t pk_min3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

struct SubsetShared {
    uint32_t lo_bits, hi_bits;                 // range of the quotients that get codes of their own
    uint32_t bucket_lo, bucket_hi, longest;
};

// LDS of the kernel (byte offsets), all of it in the dynamic part (the limit of that part is raised to all there is).  G sets share a wave: 64 / G lanes of two entries each.
struct SubsetLds {
    uint32_t shared_off, q_off, query_off, hi_off, t_off, B_off, P_off, run_off, row_off, total;
    __host__ __device__ static SubsetLds make(int L, int k, int G, int waves, bool rows_in_lds) {
        SubsetLds s;
        size_t off = 0;
        s.shared_off = 0;
        off = align_up(sizeof(SubsetShared), 16);
        s.q_off = (uint32_t)off;                         // [k][k] rows of 64 / G dwords
        off += (size_t)k * k * (64 / G) * 4;
        s.query_off = (uint32_t)off;                     // [k][128 / G] dwords
        off += (size_t)k * (128 / G) * 4;
        s.P_off = (uint32_t)(off = align_up(off, 16));
        off += (align_up((size_t)L, 64) + 1) * 8;        // written 64 at a time
        s.t_off = (uint32_t)(off = align_up(off, 16));
        off += (size_t)L * 4;
        s.B_off = (uint32_t)(off = align_up(off, 16));
        off += (size_t)k * k * 4;
        s.hi_off = (uint32_t)off;
        off += (size_t)k * (L + 1);
        s.run_off = (uint32_t)(off = align_up(off, 16));
        off += (size_t)waves * run_dwords(G) * 4;
        s.row_off = (uint32_t)(off = align_up(off, 16));
        if (rows_in_lds) off += ((size_t)k << (k - 1)) * (size_t)((L + 1) / 2) * 4;
        s.total = (uint32_t)align_up(off, 16);
        return s;
    }
};

// dwords of the rows of an instance in global memory, a multiple of 256 bytes
__host__ __device__ inline uint32_t row_dwords(int k, int rd) { return (((uint32_t)k << (k - 1)) * (uint32_t)rd + 63u) & ~63u; }

// Rows A[R' + j][j] of every set R' of C nodes (C >= 1) and every j outside it.
template <int C, int G>
__device__ __forceinline__ void subset_level(int k, int rd, int lane, int wave, int waves, const uint32_t* __restrict__ q32,
                                             const uint32_t* __restrict__ query, uint32_t* __restrict__ run32, uint32_t* rows,
                                             int run_top) {
    constexpr int kLanes = 64 / G, kPitch = 64 / G;
    const int hl = lane & (kLanes - 1), part = lane / kLanes;
    const int hload = hl < rd ? hl : rd - 1;   // lanes beyond a row read its last dword; their quotients are +inf
    const uint32_t all = (1u << k) - 1u;
    const uint32_t nsets = kSets.choose[k][C];
    const int first = kSets.first[C];
    for (uint32_t u = (uint32_t)wave * G; u < nsets; u += (uint32_t)waves * G) {
        uint32_t idx = u + (uint32_t)part;
        const bool mine = idx < nsets;
        if (G > 1 && !mine) idx = nsets - 1u;
        uint32_t entry = kSets.order[first + (int)idx];
        if (G == 1) entry = (uint32_t)__builtin_amdgcn_readfirstlane((int)entry);
        const uint32_t mp = entry & 0xFFFFu, first_row = entry >> 16;
        uint32_t a[C], qoff[C];
        {
            const uint32_t* arow = rows + first_row * (uint32_t)rd + (uint32_t)hload;
            uint32_t bits = mp;
#pragma unroll
            for (int m = 0; m < C; ++m) {
                qoff[m] = (uint32_t)(__ffs(bits) - 1) * (uint32_t)(k * kPitch) + (uint32_t)hl;
                bits &= bits - 1u;
                a[m] = arow[m * rd];
            }
        }
        uint32_t jb = all & ~mp;
        for (int i = 0; i < k - C; ++i, jb &= jb - 1u) {
            const uint32_t j = (uint32_t)__ffs(jb) - 1u;
            const uint2 qd = *reinterpret_cast<const uint2*>(query + j * (2 * kLanes) + 2 * hl);
            uint32_t v;
            {
                uint32_t x[C];
#pragma unroll
                for (int m = 0; m < C; ++m) x[m] = pk_max(q32[qoff[m] + j * kPitch], a[m]);
                v = x[0];
#pragma unroll
                for (int m = 1; m + 1 < C; m += 2) v = pk_min3(v, x[m], x[m + 1]);
                if (C % 2 == 0) v = pk_min(v, x[C - 1]);
            }
            // minima over runs of 2^r entries starting at each entry; a run that passes the end of the row holds
            // whatever lies there and is never asked for (wave shift left by one: lane i reads lane i + 1)
            run32[lane] = v;
            const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xF, 0xF, true);
            uint32_t cur = pk_min(v, (v >> 16) | (next << 16));
            run32[64 + lane] = cur;
            const uint32_t up1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x130, 0xF, 0xF, true);
            cur = pk_min(cur, up1);
            run32[128 + lane] = cur;
            const uint32_t s1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x130, 0xF, 0xF, true);
            const uint32_t up2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)s1, 0x130, 0xF, 0xF, true);
            cur = pk_min(cur, up2);
            run32[192 + lane] = cur;
            for (int r = 4; r <= run_top; ++r) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                cur = pk_min(cur, run32[(r - 1) * 64 + lane + (1 << (r - 2))]);
                run32[r * 64 + lane] = cur;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const unsigned char* runb = reinterpret_cast<const unsigned char*>(run32) + part * (kLanes * 4);
            uint32_t res[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t d = h ? qd.y : qd.x;
                const uint32_t r1 = *reinterpret_cast<const uint16_t*>(runb + (d & 0xFFFFu));
                const uint32_t r2 = *reinterpret_cast<const uint16_t*>(runb + (d >> 16));
                res[h] = r1 < r2 ? r1 : r2;
            }
            if (hl < rd && mine)   // a byte offset of 32 bits
                *reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(rows) +
                                             ((row_of(first_row, mp, j) * (uint32_t)rd + (uint32_t)hl) << 2)) = res[0] | (res[1] << 16);
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Codes with (nearly) one quotient value each, for searches whose levels are launches of their own: these cannot be
// repeated from the device, and one workgroup repeating them alone costs more than all else (with one code to 1/2048 of
// an octave that was one instance in six at L = 100, k = 10: 276 us for 64 of them, see launch_subset_solve).
// A counting sort by kRankBuckets buckets of the bit pattern, then a quotient's code is its bucket's first position plus
// the number of smaller quotients in the bucket.  Buckets of more than kRankScan quotients (ties, mostly) keep one code:
// if beta* falls into one that holds different values, the search is repeated after all.
constexpr int kRankBuckets = 8192, kRankScan = 32;
constexpr int kRankThreads = 1024;
__host__ __device__ constexpr size_t rank_scratch_bytes(int L, int k) {   // bucket ends, values, sums of the waves
    return ((size_t)kRankBuckets + (size_t)(k * (k - 1) / 2) * (size_t)(L > 1 ? L - 1 : 0) + 16u) * 4u;
}
__device__ inline void rank_quotients(int L, int k, int entries, uint32_t lo_bits, uint32_t hi_bits, const float* t_s,
                                      const float* B_s, uint16_t* q16, uint32_t* scratch) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, len = L - 1, nq = k * (k - 1) / 2 * len;
    uint32_t* ends = scratch;
    uint32_t* sums = scratch + kRankBuckets;
    uint32_t* sorted = sums + 16;
    const uint32_t span = hi_bits - lo_bits;
    const int shift = span < (uint32_t)kRankBuckets ? 0 : 32 - __clz(span / (uint32_t)kRankBuckets);
    for (int i = tid; i < kRankBuckets; i += kRankThreads) ends[i] = 0u;
    __syncthreads();
    // quotient `idx` of the unordered pairs, as in the other tables: pairs in row-major order, then layers
    auto bits_of = [&](int idx) -> uint32_t {
        const int p = idx / len, i = idx - p * len;
        int a = 0, rem = p;
        while (rem >= k - 1 - a) { rem -= k - 1 - a; ++a; }
        return __float_as_uint(__fdiv_rn(t_s[i], B_s[a * k + a + 1 + rem]));
    };
    auto ranked = [&](uint32_t bits) -> bool { return bits != 0u && bits >= lo_bits && bits <= hi_bits; };
    for (int idx = tid; idx < nq; idx += kRankThreads) {
        const uint32_t bits = bits_of(idx);
        if (ranked(bits)) atomicAdd(&ends[(bits - lo_bits) >> shift], 1u);
    }
    __syncthreads();
    // exclusive sums of the counts: eight buckets a thread
    constexpr int kEach = kRankBuckets / kRankThreads;
    uint32_t own = 0;
    for (int i = 0; i < kEach; ++i) own += ends[tid * kEach + i];
    uint32_t upto = own;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)upto, off, 64);
        upto += lane >= off ? o : 0u;
    }
    if (lane == 63) sums[wave] = upto;
    __syncthreads();
    uint32_t before = upto - own;
    for (int w = 0; w < wave; ++w) before += sums[w];
    for (int i = 0; i < kEach; ++i) {
        const uint32_t c = ends[tid * kEach + i];
        ends[tid * kEach + i] = before;
        before += c;
    }
    __syncthreads();
    for (int idx = tid; idx < nq; idx += kRankThreads) {
        const uint32_t bits = bits_of(idx);
        if (ranked(bits)) sorted[atomicAdd(&ends[(bits - lo_bits) >> shift], 1u)] = bits;
    }
    __syncthreads();   // ends[b] is now the end of bucket b, which is where bucket b + 1 starts
    for (int idx = tid; idx < k * k * entries; idx += kRankThreads) {
        const int e = idx & (entries - 1), jj = idx / entries, a = jj / k, b = jj - a * k;
        uint32_t c = kCodeInf;
        if (a != b && e >= 1 && e <= len) {
            const uint32_t bits = __float_as_uint(__fdiv_rn(t_s[e - 1], B_s[jj]));
            if (bits == 0u || bits < lo_bits) {
                c = kCodeZero;
            } else if (bits <= hi_bits) {
                const uint32_t bucket = (bits - lo_bits) >> shift;
                const uint32_t from = bucket ? ends[bucket - 1u] : 0u, to = ends[bucket];
                uint32_t smaller = 0;
                if (to - from <= (uint32_t)kRankScan)
                    for (uint32_t i = from; i < to; ++i) smaller += sorted[i] < bits ? 1u : 0u;
                c = kCodeZero + 1u + from + smaller;
            }
        }
        q16[idx] = (uint16_t)c;
    }
    __syncthreads();
}
static_assert(kCodeZero + 1 + (PPO_MAX_K * (PPO_MAX_K - 1) / 2) * (PPO_MAX_L - 1) < kCodeInf, "ranks stay below +inf");

}  // namespace

constexpr int kSubsetMaxWaves = 16;
static_assert(kRankThreads == kSubsetMaxWaves * 64, "searches that rank their quotients run with all the waves");

// KMAX: the most nodes an instantiation takes.  Up to 8 of them 64 registers hold a set's rows, and a compute unit
// holds 32 waves (two workgroups of 16, or four of 8); beyond that 80 registers and 24 waves.
constexpr int kSmallK = 8;

// Part of the search a launch does: all of it, or (many nodes: the levels are launches of their own, see
// launch_subset_solve) the tables and the rows of the sets of one node, or what follows the last level.  Between those
// launches the tables lie behind an instance's rows, as an image of this kernel's LDS.
enum { kWhole = 0, kTablesOnly = 1, kAfterLevels = 2 };

template <int G, int KMAX, bool LDSROWS, int PART>
__global__ __launch_bounds__(kSubsetMaxWaves * 64, KMAX <= kSmallK ? 8 : 6) void subset_solve_kernel(
    const float* __restrict__ t_in, const float* __restrict__ m_in, const float* __restrict__ M_in,
    const float* __restrict__ B_in, int L, int k, int n_inst, float* __restrict__ beta_out, int32_t* __restrict__ cuts_out,
    int32_t* __restrict__ order_out, uint32_t* row_slots, uint32_t slot_dwords) {
    extern __shared__ __align__(16) unsigned char sm[];
    const int tid = threadIdx.x, threads = blockDim.x, lane = tid & 63, waves = threads >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SubsetLds lds = SubsetLds::make(L, k, G, waves, LDSROWS);
    constexpr int kEntries = 128 / G;
    const int rd = (L + 1) / 2;
    SubsetShared& sh = *reinterpret_cast<SubsetShared*>(sm + lds.shared_off);
    uint16_t* q16 = reinterpret_cast<uint16_t*>(sm + lds.q_off);
    uint32_t* query = reinterpret_cast<uint32_t*>(sm + lds.query_off);
    double* P = reinterpret_cast<double*>(sm + lds.P_off);
    float* t_s = reinterpret_cast<float*>(sm + lds.t_off);
    float* B_s = reinterpret_cast<float*>(sm + lds.B_off);
    unsigned char* hi_s = sm + lds.hi_off;
    uint32_t* run32 = reinterpret_cast<uint32_t*>(sm + lds.run_off) + wave * run_dwords(G);
    uint32_t* rows = LDSROWS ? reinterpret_cast<uint32_t*>(sm + lds.row_off) : row_slots + (size_t)blockIdx.x * slot_dwords;
    const uint32_t all = (1u << k) - 1u;
    if (lane < 48) run32[run_levels(G) * 64 + lane] = kCodeInf | (kCodeInf << 16);

    for (uint32_t inst = blockIdx.x; inst < (uint32_t)n_inst; inst += gridDim.x) {
        uint4* image = reinterpret_cast<uint4*>(rows + row_dwords(k, rd));
        if (PART == kAfterLevels) {
            for (uint32_t i = (uint32_t)tid; i < lds.run_off / 16u; i += (uint32_t)threads)
                reinterpret_cast<uint4*>(sm)[i] = image[i];
            __syncthreads();
        }
        bool levels_done = PART == kAfterLevels;
        if (PART != kAfterLevels) {   // (not indented: the whole of the tables)
        // inputs; a transfer size of zero is +0 whatever its sign bit says
        float* m_s = reinterpret_cast<float*>(run32 - wave * run_dwords(G));   // the run tables are not in use yet
        for (int i = tid; i < L; i += threads) {
            const float x = t_in[(size_t)inst * L + i];
            t_s[i] = x == 0.0f ? 0.0f : x;
            m_s[i] = m_in[(size_t)inst * L + i];
        }
        for (int i = tid; i < k * k; i += threads) {
            const int a = i / k, b = i - a * k;   // the element with the smaller row index is the one read
            B_s[i] = B_in[(size_t)inst * k * k + (a < b ? i : b * k + a)];
        }
        if (tid == 0) sh.longest = 0u;
        __syncthreads();
        if (wave == 0) {
            // prefix sums in index order in binary64 (the definition fixes the order)
            // (a lane's weight is fetched from its register: no memory access in the chain of additions; all lanes add
            // and store the same: a store by one lane took 4096 x (96, 8) from 612 to 634 us)
            double acc = 0.0;
            P[0] = 0.0;
            for (int base = 0; base < L; base += 64) {
                const float w = base + lane < L ? m_s[base + lane] : 0.0f;
#pragma unroll
                for (int i = 0; i < 64; ++i) {
                    acc = acc + (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), i));
                    P[base + i + 1] = acc;
                }
            }
        }
        if (wave == waves - 1) {
            // range of the quotients: a correctly rounded division is monotone in both operands
            float tmin = __uint_as_float(kInfBits), tmax = 0.0f, bmin = __uint_as_float(kInfBits), bmax = 0.0f;
            for (int i = lane; i < L - 1; i += 64) {
                const float x = t_s[i];
                tmax = x > tmax ? x : tmax;
                tmin = x != 0.0f && x < tmin ? x : tmin;
            }
            for (int i = lane; i < k * k; i += 64) {
                const float x = B_s[i];
                if (i / k != i % k) {
                    bmin = x < bmin ? x : bmin;
                    bmax = x > bmax ? x : bmax;
                }
            }
            for (int off = 32; off >= 1; off >>= 1) {
                const float a = __shfl_xor(tmin, off, 64), b = __shfl_xor(tmax, off, 64);
                const float c = __shfl_xor(bmin, off, 64), d = __shfl_xor(bmax, off, 64);
                tmin = a < tmin ? a : tmin;
                tmax = b > tmax ? b : tmax;
                bmin = c < bmin ? c : bmin;
                bmax = d > bmax ? d : bmax;
            }
            if (lane == 0) {
                // no quotient but 0 (or none at all): any range will do
                const bool some = tmax > 0.0f && bmax > 0.0f;
                const uint32_t lo = some ? __float_as_uint(__fdiv_rn(tmin, bmax)) : 0u;
                const uint32_t hi = some ? __float_as_uint(__fdiv_rn(tmax, bmin)) : 0u;
                sh.lo_bits = lo < kInfBits ? lo : kInfBits - 1u;
                sh.hi_bits = hi < kInfBits ? hi : kInfBits - 1u;
            }
        }
        __syncthreads();
        // hi[j][e]: the window's length does not shrink when its end is moved back (sums of weights >= 0), so a binary
        // search finds what a scan would.  Window queries: (e, min(hi, L-1)] is covered by two runs of 2^r entries, the
        // one that starts at e + 1 and the one that ends at its end; the table holds their byte offsets.
        int longest = 0;
        for (int idx = tid; idx < k * kEntries; idx += threads) {
            const int j = idx / kEntries, e = idx - j * kEntries;
            uint32_t d = no_window(G) | (no_window(G) << 16);
            if (e < L) {
                const double cap = (double)M_in[(size_t)inst * k + j], from = P[e];
                int good = e, step = 1;
                while (step < L) step <<= 1;
                for (; step >= 1; step >>= 1) {
                    const int e2 = good + step;
                    if (e2 <= L && P[e2] - from <= cap) good = e2;
                }
                hi_s[j * (L + 1) + e] = (unsigned char)good;
                const int top = good < L - 1 ? good : L - 1;
                if (top > e) {
                    int r = 31 - __clz(top - e);
                    r = r > run_levels(G) - 1 ? run_levels(G) - 1 : r;
                    // rows of a wave's run table are 64 dwords, G sets side by side
                    d = (uint32_t)(r * 256 + (e + 1) * 2) | ((uint32_t)(r * 256 + (top - (1 << r) + 1) * 2) << 16);
                    longest = r > longest ? r : longest;
                }
            }
            query[idx] = d;
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const int o = __shfl_xor(longest, off, 64);
            longest = o > longest ? o : longest;
        }
        if (lane == 0) atomicMax(&sh.longest, (uint32_t)longest);
        if (tid < k) hi_s[tid * (L + 1) + L] = (unsigned char)L;
        __syncthreads();
        }
        const int run_top = (int)sh.longest;

        uint32_t best = kCodeInf, best_bits = kInfBits;
        for (;;) {
            const uint32_t lo_bits = sh.lo_bits, hi_bits = sh.hi_bits;
            const uint32_t span = hi_bits - lo_bits;
            const int shift = span < kFinestCodes ? 0 : 32 - __clz(span / kFinestCodes);
            auto code_of = [&](uint32_t bits) -> uint32_t {
                if (bits == 0u || bits < lo_bits) return kCodeZero;
                if (bits > hi_bits) return kCodeInf;
                return kCodeZero + 1u + ((bits - lo_bits) >> shift);
            };
            if (!levels_done) {
            // quotients of every ordered pair of nodes (Eq. 3): entry e of the row of (j, j'') belongs to the cut e
            if (PART == kTablesOnly) {
                rank_quotients(L, k, kEntries, lo_bits, hi_bits, t_s, B_s, q16, reinterpret_cast<uint32_t*>(sm + lds.row_off));
            } else {
                for (int idx = tid; idx < k * k * kEntries; idx += threads) {
                    const int e = idx & (kEntries - 1), jj = idx / kEntries, a = jj / k, b = jj - a * k;
                    uint32_t c = kCodeInf;
                    if (a != b && e >= 1 && e <= L - 1) c = code_of(__float_as_uint(__fdiv_rn(t_s[e - 1], B_s[jj])));
                    q16[idx] = (uint16_t)c;
                }
            }
            // sets of one node: its segment runs to the end of the chain
            for (int idx = tid; idx < k * rd; idx += threads) {
                const int j = idx / rd, d = idx - j * rd, e = 2 * d;
                const uint32_t v0 = hi_s[j * (L + 1) + e] == L ? kCodeZero : kCodeInf;
                const uint32_t v1 = e + 1 < L && hi_s[j * (L + 1) + e + 1] == L ? kCodeZero : kCodeInf;
                rows[row_of(0u, 0u, (uint32_t)j) * (uint32_t)rd + (uint32_t)d] = v0 | (v1 << 16);
            }
            if (tid == 0) {
                sh.bucket_lo = ~0u;
                sh.bucket_hi = 0u;
            }
            __syncthreads();
            if (PART == kTablesOnly) break;
            const uint32_t* q32 = reinterpret_cast<const uint32_t*>(q16);
#define PPO_SUBSET_LEVEL(C_)                                                                            \
    if (C_ < KMAX && k > C_) {                                                                          \
        subset_level<C_, G>(k, rd, lane, wave, waves, q32, query, run32, rows, run_top);                \
        __syncthreads();                                                                                \
    }
            PPO_SUBSET_LEVEL(1)
            PPO_SUBSET_LEVEL(2)
            PPO_SUBSET_LEVEL(3)
            PPO_SUBSET_LEVEL(4)
            PPO_SUBSET_LEVEL(5)
            PPO_SUBSET_LEVEL(6)
            PPO_SUBSET_LEVEL(7)
            PPO_SUBSET_LEVEL(8)
            PPO_SUBSET_LEVEL(9)
            PPO_SUBSET_LEVEL(10)
            PPO_SUBSET_LEVEL(11)
#undef PPO_SUBSET_LEVEL
            }
            levels_done = false;
            // the full set's rows are the last k ones
            const uint32_t full_row = ((uint32_t)k << (k - 1)) - (uint32_t)k;
            best = lane < k ? rows[(full_row + (uint32_t)lane) * (uint32_t)rd] & 0xFFFFu : kCodeInf;
            for (int off = 8; off >= 1; off >>= 1) {
                const uint32_t o = (uint32_t)__shfl_xor((int)best, off, 64);
                best = o < best ? o : best;
            }
            best = (uint32_t)__builtin_amdgcn_readfirstlane((int)best);
            if (best >= kCodeInf) break;
            if (best == kCodeZero) {   // the optimum is 0 (after the first pass it lies in the range)
                best_bits = 0u;
                break;
            }
            uint32_t least = ~0u, most = 0u;
            for (int idx = tid; idx < k * k * kEntries; idx += threads) {
                const int e = idx & (kEntries - 1), jj = idx / kEntries;
                if (q16[idx] == best) {
                    const uint32_t bits = __float_as_uint(__fdiv_rn(t_s[e - 1], B_s[jj]));
                    least = bits < least ? bits : least;
                    most = bits > most ? bits : most;
                }
            }
            if (least != ~0u) {
                atomicMin(&sh.bucket_lo, least);
                atomicMax(&sh.bucket_hi, most);
            }
            __syncthreads();
            const uint32_t from = sh.bucket_lo, to = sh.bucket_hi;
            if (from >= to) {
                best_bits = from;
                break;
            }
            if (tid == 0) {
                sh.lo_bits = from;
                sh.hi_bits = to;
            }
            __syncthreads();
        }

        if (PART == kTablesOnly) {
            for (uint32_t i = (uint32_t)tid; i < lds.run_off / 16u; i += (uint32_t)threads)
                image[i] = reinterpret_cast<const uint4*>(sm)[i];
            __syncthreads();
            continue;
        }

        // The lexicographically smallest optimal ordering, position by position: F = cuts that the chosen prefix reaches
        // with all its links at most beta*, G_j = those of F whose link into candidate j is at most beta*.  A candidate
        // completes to an optimum iff A[unused][j][e] <= beta* for some e in G_j; the smallest such node is taken, and F
        // for the next position is the set of cuts that a window of that node starting in G_j covers (hi[j][.] does not
        // decrease, so the latest start below a cut decides).
        auto hi = [&](int j, int e) -> int { return hi_s[j * (L + 1) + e]; };
        auto covered = [&](unsigned long long g0, unsigned long long g1, int j, int e2) -> bool {
            unsigned long long m0 = g0, m1 = 0;
            if (e2 < 64)
                m0 = g0 & ((1ull << e2) - 1ull);
            else
                m1 = e2 >= 128 ? g1 : g1 & ((1ull << (e2 - 64)) - 1ull);
            const int from = m1 ? 127 - __clzll((long long)m1) : m0 ? 63 - __clzll((long long)m0) : -1;
            return from >= 0 && hi(j, from) >= e2;
        };
        int32_t* cuts = cuts_out + (size_t)inst * (k - 1);
        int32_t* order = order_out + (size_t)inst * k;
        const bool feasible = best < kCodeInf && best_bits < kInfBits;
        if (!feasible) {
            if (tid == 0) beta_out[inst] = __uint_as_float(kInfBits);
            if (tid < k) order[tid] = -1;
            if (tid < k - 1) cuts[tid] = -1;
        } else if (wave == 0) {
            // One wave: the other workgroups of the compute unit go on meanwhile, and a position costs about as many
            // instructions as a row.  Four candidates at a time, so that their rows are in flight together.
            constexpr int kHalves = G == 1 ? 2 : 1;
            const uint16_t* rows16 = reinterpret_cast<const uint16_t*>(rows);
            const int ec[2] = {lane < L ? lane : L - 1, lane + 64 < L ? lane + 64 : L - 1};
            unsigned long long F[2] = {1ull, 0ull};   // the first segment starts at 0
            unsigned long long my_start[2] = {0ull, 0ull};   // lane s: G of the node at position s
            uint32_t unused = all, first_row = ((uint32_t)k << (k - 1)) - (uint32_t)k;   // first row of `unused`
            int last = 0, my_node = 0;
            for (int s = 0; s < k; ++s) {
                int chosen = -1;
                unsigned long long Gc[2] = {0ull, 0ull};
                for (uint32_t jb = unused; jb && chosen < 0;) {
                    int js[4];
                    uint32_t av[4][kHalves], qv[4][kHalves];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        js[c] = jb ? __ffs(jb) - 1 : js[c > 0 ? c - 1 : 0];
                        jb &= jb - 1u;
                        const uint32_t row = first_row + (uint32_t)__popc(unused & ((1u << js[c]) - 1u));
#pragma unroll
                        for (int h = 0; h < kHalves; ++h) {
                            av[c][h] = rows16[row * (uint32_t)(2 * rd) + (uint32_t)ec[h]];
                            qv[c][h] = q16[(last * k + js[c]) * kEntries + ec[h]];
                        }
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        unsigned long long g[2] = {0ull, 0ull}, ok = 0ull;
#pragma unroll
                        for (int h = 0; h < kHalves; ++h) {
                            // beyond the first position F holds no cut 0
                            const bool in_g = ((F[h] >> lane) & 1ull) && (s == 0 || qv[c][h] <= best);
                            g[h] = __ballot(in_g);
                            ok |= __ballot(in_g && av[c][h] <= best);
                        }
                        if (ok && chosen < 0) {
                            chosen = js[c];
                            Gc[0] = g[0];
                            Gc[1] = g[1];
                        }
                    }
                }
                if (chosen < 0) chosen = __ffs(unused) - 1;   // cannot happen: some completion of the prefix reaches the optimum
                if (lane == s) {
                    my_node = chosen;
                    my_start[0] = Gc[0];
                    my_start[1] = Gc[1];
                }
                F[0] = __ballot(lane >= 1 && lane < L && covered(Gc[0], Gc[1], chosen, lane));
                if (G == 1) F[1] = __ballot(lane + 64 < L && covered(Gc[0], Gc[1], chosen, lane + 64));
                unused &= ~(1u << chosen);
                first_row -= row_of(0u, unused, (uint32_t)chosen) - (uint32_t)__popc(unused & ((1u << chosen) - 1u));
                last = chosen;
            }
            // cuts, latest segment first: each time the smallest start (reached by the prefix, link at most beta*) whose
            // window covers the end
            int e = L;
            for (int s = k - 1; s >= 1; --s) {
                const int js = __builtin_amdgcn_readlane(my_node, s);
                unsigned long long start[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    start[h] = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_start[h], s) |
                               ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_start[h] >> 32), s) << 32);
                const unsigned long long m0 = __ballot(((start[0] >> lane) & 1ull) && lane < e && hi(js, ec[0]) >= e);
                unsigned long long m1 = 0ull;
                if (G == 1) m1 = __ballot(((start[1] >> lane) & 1ull) && lane + 64 < e && hi(js, ec[1]) >= e);
                const int first = m0 ? __ffsll((long long)m0) - 1 : 63 + __ffsll((long long)m1);
                if (lane == 0) cuts[s - 1] = (int32_t)first;
                e = first;
            }
            if (lane == 0) beta_out[inst] = __uint_as_float(best_bits);
            if (lane < k) order[lane] = my_node;
        }
        __syncthreads();   // the next instance overwrites what the last steps read
    }
}

// One level of the sets over many workgroups: grid.x of them per instance, grid.y = instance.
template <int G, int C>
__global__ __launch_bounds__(512, 6) void subset_level_kernel(int L, int k, uint32_t* row_slots, uint32_t slot_dwords,
                                                              uint32_t image_off) {
    extern __shared__ __align__(16) unsigned char sm[];
    const int tid = threadIdx.x, lane = tid & 63, waves = blockDim.x >> 6, rd = (L + 1) / 2;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t* rows = row_slots + (size_t)blockIdx.y * slot_dwords;
    const uint4* image = reinterpret_cast<const uint4*>(rows + row_dwords(k, rd)) + image_off / 16u;
    const uint32_t tables16 = (uint32_t)(k * k * (64 / G) + k * (128 / G)) / 4u;
    for (uint32_t i = (uint32_t)tid; i < tables16; i += blockDim.x) reinterpret_cast<uint4*>(sm)[i] = image[i];
    const uint32_t* q32 = reinterpret_cast<const uint32_t*>(sm);
    uint32_t* run32 = reinterpret_cast<uint32_t*>(sm) + tables16 * 4u + (uint32_t)wave * run_dwords(G);
    if (lane < 48) run32[run_levels(G) * 64 + lane] = kCodeInf | (kCodeInf << 16);
    __syncthreads();
    const SubsetShared& sh = *reinterpret_cast<const SubsetShared*>(rows + row_dwords(k, rd));
    subset_level<C, G>(k, rd, lane, (int)blockIdx.x * waves + wave, (int)gridDim.x * waves, q32,
                       q32 + k * k * (64 / G), run32, rows, (int)sh.longest);
}

// Bytes of rows in global memory that one workgroup of the kernel needs; 0 if its rows stay in LDS, which they do while
// two workgroups fit a compute unit's.
namespace {
int subset_sets_per_wave(int L) { return L <= 64 ? 2 : 1; }
// as many waves as the widest level can use: 16 if it keeps them busy twice, else up to 8
int subset_waves(int L, int k) {
    const int G = subset_sets_per_wave(L);
    const int widest = ((int)kSetsHost.choose[k][k / 2] + G - 1) / G;
    return widest < 2 ? 2 : widest >= 2 * kSubsetMaxWaves ? kSubsetMaxWaves : widest > 8 ? 8 : widest;
}
}  // namespace

size_t subset_slot_bytes(int L, int k) {
    if (k <= kSmallK) {
        const SubsetLds s = SubsetLds::make(L, k, subset_sets_per_wave(L), subset_waves(L, k), true);
        if (2u * s.total <= (uint32_t)kLdsBytesPerCU) return 0;
    }
    const SubsetLds s = SubsetLds::make(L, k, subset_sets_per_wave(L), 1, false);
    return (size_t)row_dwords(k, (L + 1) / 2) * 4 + align_up(s.run_off, 256);
}

// Launches of the levels of up to `cnt` instances whose tables are in place.
template <int G, int C>
static hipError_t launch_level(int L, int k, int cnt, uint32_t* slots, size_t slot, uint32_t image_off, hipStream_t stream) {
    if constexpr (C < PPO_MAX_K) {
        if (C >= k) return hipSuccess;
        constexpr int kWaves = 8;   // three workgroups to a compute unit, with 80 registers
        const size_t lds = (size_t)(k * k * (64 / G) + k * (128 / G)) * 4 + (size_t)kWaves * run_dwords(G) * 4;
        static std::atomic<uint64_t> lds_allowed{0};
        hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&subset_level_kernel<G, C>), lds_allowed);
        if (e != hipSuccess) return e;
        const uint32_t most = (kSetsHost.choose[k][C] + (uint32_t)(kWaves * G) - 1u) / (uint32_t)(kWaves * G);
        const uint32_t cap = (768u + (uint32_t)cnt - 1u) / (uint32_t)cnt;
        hipLaunchKernelGGL((subset_level_kernel<G, C>), dim3(most < cap ? most : cap, cnt), dim3(kWaves * 64), lds, stream, L, k,
                           slots, (uint32_t)(slot / 4), image_off);
        e = hipGetLastError();
        return e != hipSuccess ? e : launch_level<G, C + 1>(L, k, cnt, slots, slot, image_off, stream);
    } else {
        return hipSuccess;
    }
}

// slots: `slot_count` areas of subset_slot_bytes (unused if that is 0).  Up to kSmallK nodes a workgroup does the whole
// search and keeps its area for all its instances; with more nodes an instance has enough sets for many workgroups, and
// the levels of `slot_count` instances at a time are launches over all of them: 1 x (64, 11) 76 us against 410 in one
// workgroup, 64 x (100, 10) 133 against 358, 37 x (127, 9) 87 against 174.
hipError_t launch_subset_solve(const float* t, const float* m, const float* M, const float* B, int L, int k, int n_inst,
                               float* beta_out, int32_t* cuts_out, int32_t* order_out, void* slots, size_t slot_count,
                               hipStream_t stream) {
    const int G = subset_sets_per_wave(L);
    const size_t slot = subset_slot_bytes(L, k);
    if (bands_apply(L, k, n_inst, slot, slot_count))
        return launch_bands_solve(t, m, M, B, L, k, n_inst, beta_out, cuts_out, order_out, slots, slot, slot_count, stream);
    if (slot != 0 && slot_count > (size_t)n_inst) slot_count = (size_t)n_inst;
    auto launch = [&](auto kernel, std::atomic<uint64_t>& lds_allowed, int first, int cnt, uint32_t grid, int part = kWhole) -> hipError_t {
        const int waves = k > kSmallK ? kSubsetMaxWaves : subset_waves(L, k);
        SubsetLds s = SubsetLds::make(L, k, G, waves, slot == 0);
        if (part == kTablesOnly) s.total += (uint32_t)rank_scratch_bytes(L, k);
        const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(kernel), lds_allowed);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * 64), s.total, stream, t + (size_t)first * L, m + (size_t)first * L,
                           M + (size_t)first * k, B + (size_t)first * k * k, L, k, cnt, beta_out + first,
                           cuts_out + (size_t)first * (k - 1), order_out + (size_t)first * k, static_cast<uint32_t*>(slots),
                           (uint32_t)(slot / 4));
        return hipGetLastError();
    };
    static std::atomic<uint64_t> allowed[8];
    if (slot == 0) {
        // a workgroup per instance; a launch may have fewer than 2^32 threads, which 4.2 million workgroups of 1024 are not
        constexpr int kMost = 1 << 20;
        for (int first = 0;; first += kMost) {
            const int left = n_inst - first, cnt = left < kMost ? left : kMost;
            const hipError_t e = G == 2 ? launch(&subset_solve_kernel<2, kSmallK, true, kWhole>, allowed[0], first, cnt, (uint32_t)cnt)
                                        : launch(&subset_solve_kernel<1, kSmallK, true, kWhole>, allowed[1], first, cnt, (uint32_t)cnt);
            if (e != hipSuccess || cnt == left) return e;
        }
    }
    if (k <= kSmallK)
        return G == 2 ? launch(&subset_solve_kernel<2, kSmallK, false, kWhole>, allowed[2], 0, n_inst, (uint32_t)slot_count)
                      : launch(&subset_solve_kernel<1, kSmallK, false, kWhole>, allowed[3], 0, n_inst, (uint32_t)slot_count);
    const uint32_t image_off = SubsetLds::make(L, k, G, 1, false).q_off;
    for (int first = 0; first < n_inst; first += (int)slot_count) {
        const int cnt = n_inst - first < (int)slot_count ? n_inst - first : (int)slot_count;
        hipError_t e = G == 2 ? launch(&subset_solve_kernel<2, PPO_MAX_K, false, kTablesOnly>, allowed[4], first, cnt, (uint32_t)cnt, kTablesOnly)
                              : launch(&subset_solve_kernel<1, PPO_MAX_K, false, kTablesOnly>, allowed[5], first, cnt, (uint32_t)cnt, kTablesOnly);
        if (e != hipSuccess) return e;
        e = G == 2 ? launch_level<2, 1>(L, k, cnt, static_cast<uint32_t*>(slots), slot, image_off, stream)
                   : launch_level<1, 1>(L, k, cnt, static_cast<uint32_t*>(slots), slot, image_off, stream);
        if (e != hipSuccess) return e;
        e = G == 2 ? launch(&subset_solve_kernel<2, PPO_MAX_K, false, kAfterLevels>, allowed[6], first, cnt, (uint32_t)cnt)
                   : launch(&subset_solve_kernel<1, PPO_MAX_K, false, kAfterLevels>, allowed[7], first, cnt, (uint32_t)cnt);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ppo
