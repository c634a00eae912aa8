// Cluster form of the exact search: the hosting nodes are a sequence of p distinct nodes chosen from a
// cluster of n, and p itself is free (1 <= p <= pmax).  In the paper the partitioner fixes the number of
// partitions and the placement picks that many nodes out of the communication graph as a simple path
// (Sec. III-B1/2); its evaluation uses clusters of 5 to 50 devices (Sec. IV).
//
// The bottleneck of Eq. 2 is a maximum over links, so what is still to be paid from a cut on depends only
// on the node that takes the next segment, the cut, and the set R of nodes not used before it:
//     A[R][j][e]     = min over e' in (e, L] with layers [e, e') fitting node j      of  rest[R \ j][j][e']
//     rest[R'][j][e'] = 0                                                   if e' = L
//                     = min over j'' in R' of max(q_{j,j''}[e'-1], A[R'][j''][e'])   if another segment may
//                                                                            follow (n - |R'| < pmax)
//                     = +inf                                                otherwise
// (q_{a,b}[i] = t[i] / B[a][b], Eq. 3) and beta* = min over j of A[All][j][0].  Rows are computed level by
// level in |R|, one launch per level, one wave per row, on 16-bit order codes of the quotients.  The
// lexicographically smallest optimal sequence (a sequence before its extensions) is rebuilt position by
// position from the cuts the prefix reaches within beta* and the rows of A, then the cuts by the fixed-k cut rule.
// Where it pays, the search runs on the nodes and cuts that can matter alone (ppo_cluster_bound.hip); the kernels after it
// take an instance's own number of nodes and layers from its tables.
#include <array>
#include <utility>

#include "ppo_cluster.h"

namespace ppo {

// Row number of A[R][j], j in R: the rows of the sets before R in numeric order (the sum of their sizes),
// then the members of R in increasing order.  The sum of the sizes of all sets below R: a member b of R
// with h members above it stands for the 2^b sets that agree with R above b and lack b; they have
// h + (a free choice below b) members: h 2^b + b 2^(b-1) in all (b 2^(b-1) written (b << b) >> 1: no case for b = 0).
__host__ __device__ inline uint32_t cluster_first_row(uint32_t R, int n) {
    uint32_t rows = 0, above = 0;
    for (int b = n - 1; b >= 0; --b) {
        if (!((R >> b) & 1u)) continue;
        rows += (above << b) + (((uint32_t)b << b) >> 1);
        ++above;
    }
    return rows;
}
size_t cluster_tables_bytes(int L, int n) { return ClusterLayout::make(L, n).stride; }
size_t cluster_rows_bytes(int L, int n) { return ClusterLayout::make(L, n).rows_bytes(); }

// ---------------------------------------------------------------------------------------------
// Tables of one instance: hi[j][e] = last e' such that layers [e, e') fit node j (e if none; the memory
// rule with binary64 prefix sums) and the quotients of Eq. 3; then, in a second kernel over slices of
// the quotients, their order codes (1 + the number of strictly smaller quotients of the instance; 0 for the value 0).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kClPreThreads) void cluster_tables_kernel(const float* __restrict__ t,
                                                                      const float* __restrict__ m,
                                                                      const float* __restrict__ M,
                                                                      const float* __restrict__ B, ClusterLayout y,
                                                                      unsigned char* __restrict__ ws) {
    __shared__ double P[PPO_MAX_L + 1];
    const int L = y.L, n = y.n, inst = blockIdx.x, tid = threadIdx.x;
    const float* ti = t + (size_t)inst * L;
    const float* mi = m + (size_t)inst * L;
    const float* Mi = M + (size_t)inst * n;
    const float* Bi = B + (size_t)inst * n * n;
    unsigned char* base = ws + (size_t)inst * y.stride;
    unsigned char* hi = base + y.hi_off;
    float* dec = reinterpret_cast<float*>(base + y.dec_off);
    float* qv = reinterpret_cast<float*>(base + y.qv_off);
    if (tid == 0) {
        double acc = 0.0;
        P[0] = 0.0;
        for (int i = 0; i < L; ++i) {
            acc = acc + (double)mi[i];
            P[i + 1] = acc;
        }
        dec[0] = 0.0f;
        *reinterpret_cast<uint32_t*>(base + y.flag_off()) = 0u;
    }
    __syncthreads();
    for (int idx = tid; idx < n * (L + 1); idx += kClPreThreads) {
        const int j = idx / (L + 1), e = idx - j * (L + 1);
        const double cap = (double)Mi[j];
        int lo = e, top = L;   // the last end that fits; P does not decrease
        while (lo < top) {
            const int mid = (lo + top + 1) >> 1;
            if ((P[mid] - P[e]) <= cap) lo = mid; else top = mid - 1;
        }
        hi[idx] = (unsigned char)lo;
    }
    // The quotients of one link, t[i] / B, are in the order of the t[i] (a correctly rounded division by a
    // positive number is monotone), so each link's row is written sorted: position r holds the quotient of the
    // layer with the r-th smallest t (ties by index).  Ranking a quotient among all of them is then a binary
    // search per link instead of a comparison with every quotient.
    __shared__ float t_s[PPO_MAX_L];
    __shared__ unsigned char ord_s[PPO_MAX_L];
    for (int i = tid; i < L - 1; i += kClPreThreads) t_s[i] = ti[i] == 0.0f ? 0.0f : ti[i];   // -0 is a size of zero: +0
    __syncthreads();
    for (int i = tid; i < L - 1; i += kClPreThreads) {
        const float x = t_s[i];
        int pos = 0;
        for (int i2 = 0; i2 < L - 1; ++i2) pos += (t_s[i2] < x || (t_s[i2] == x && i2 < i)) ? 1 : 0;
        ord_s[pos] = (unsigned char)i;
        base[y.ord_off + pos] = (unsigned char)i;
    }
    __syncthreads();
    for (int idx = tid; idx < y.nq; idx += kClPreThreads) {
        const int p = idx / (L - 1), r = idx - p * (L - 1);
        int a = 0, rem = p;
        while (rem >= n - 1 - a) { rem -= n - 1 - a; ++a; }
        qv[idx] = __fdiv_rn(t_s[ord_s[r]], Bi[a * n + a + 1 + rem]);
    }
}

// Order codes: grid.x slices of 256 quotients, grid.y = instance.  All sorted rows are staged in LDS; four threads per
// quotient add up, over a quarter of the links each, how many of a link's quotients are strictly below it (a binary
// search each).  Serial searches bound it, and slices are few (75 at 20 nodes and 100 layers): one thread per quotient
// took 54 us there.
constexpr int kClCountSlice = 256, kClCountParts = 4, kClCountThreads = kClCountSlice * kClCountParts;
__global__ __launch_bounds__(kClCountThreads) void cluster_count_kernel(ClusterLayout whole, unsigned char* __restrict__ ws) {
    extern __shared__ __align__(16) float cl_rows[];   // [npairs][L-1], then the sums of the slice
    const int inst = blockIdx.y, tid = threadIdx.x;
    unsigned char* base = ws + (size_t)inst * whole.stride;
    const ClusterLayout y = cluster_layout(whole, base);
    const int L = y.L, nq = y.nq, len = L - 1;
    if ((int)blockIdx.x * kClCountSlice >= nq) return;
    const float* __restrict__ qv = reinterpret_cast<const float*>(base + y.qv_off);
    int* below_s = reinterpret_cast<int*>(cl_rows + nq);
    for (int i = tid; i < nq; i += kClCountThreads) cl_rows[i] = qv[i];
    if (tid < kClCountSlice) below_s[tid] = 0;
    __syncthreads();
    const int mine = tid & (kClCountSlice - 1), idx = blockIdx.x * kClCountSlice + mine;
    const float x = cl_rows[idx < nq ? idx : nq - 1];
    int below = 0;
    int widest = 64;
    while (widest > len) widest >>= 1;
    // four links at a time, so that four reads are in flight at every step of the searches
    for (int p0 = 4 * (tid / kClCountSlice); p0 < y.npairs; p0 += 4 * kClCountParts) {
        int pos[4] = {0, 0, 0, 0};   // number of entries of each row below x
        const float* row[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) row[u] = cl_rows + (p0 + u < y.npairs ? p0 + u : p0) * len;
        for (int step = widest; step >= 1; step >>= 1) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int np = pos[u] + step;
                v[u] = row[u][(np <= len ? np : len) - 1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int np = pos[u] + step;
                if (np <= len && v[u] < x) pos[u] = np;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) below += p0 + u < y.npairs ? pos[u] : 0;
    }
    atomicAdd(&below_s[mine], below);
    __syncthreads();
    if (tid >= kClCountSlice || idx >= nq) return;
    below = below_s[mine];
    const int p = idx / len, r = idx - p * len;
    const int i = base[y.ord_off + r];
    // a link that takes no time ties with no link at all
    reinterpret_cast<uint16_t*>(base + y.qc_off)[p * L + i] = (uint16_t)(x == 0.0f ? kClZero : kClZero + 1 + below);
    reinterpret_cast<float*>(base + y.dec_off)[1 + below] = x;
}

// ---------------------------------------------------------------------------------------------
// One level: every row A[R][j] with |R| = level.  The unit of work of a wave is a set R' with |R'| =
// level - 1 (two of them on chains of up to 63 layers, 32 lanes each): it loads the rows A[R'][j''] once (two
// entries per lane) and produces A[R' + j][j] for every j outside R'.  For each j: the `rest` row (quotients
// from a copy of the table in LDS, shifted so that entry e holds q[e-1]), then a table of minima over runs of
// 1, 2, 4 .. entries of it in LDS, as far as the longest window needs them, from which the minimum over the
// window (e, hi[j][e]] is two reads.  grid.x workgroups share the sets, grid.y = instance.
//
// What bounds it: instruction issue of all kinds.  One cluster of 20 nodes and 100 layers searched whole takes 67 scalar, 56
// vector and 21 LDS instructions a row, which fills 0.65, 0.54 and 0.46 of these units' time; of the time of its five to six waves on
// a SIMD 0.38 is spent ready and waiting for a turn, 0.32 waiting for data.  The quotients of unordered pairs and run
// tables without padding let two workgroups of 16 waves share a compute unit there (level 11: 367 us before, 340 now,
// under the profiler); two sets to a wave nearly halve the levels of 50 layers (15 nodes, 32 instances: 253 us to 137).
// ---------------------------------------------------------------------------------------------
typedef unsigned short cl_ushort2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cl_pk_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(cl_ushort2, a), __builtin_bit_cast(cl_ushort2, b)));
}
__device__ __forceinline__ uint32_t cl_pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(cl_ushort2, a), __builtin_bit_cast(cl_ushort2, b)));
}

// Binomial coefficients C(i, j), i, j <= PPO_CLUSTER_MAX_N, and the set of a given size with a given index:
// sets of c nodes are numbered by sum over their members b_c > ... > b_1 of C(b_i, i) (the combinatorial
// number system), so that the sets of one level can be dealt out evenly to the waves.
struct ClusterBinomials {
    uint32_t c[PPO_CLUSTER_MAX_N + 1][PPO_CLUSTER_MAX_N + 1];
    constexpr ClusterBinomials() : c{} {
        for (int i = 0; i <= PPO_CLUSTER_MAX_N; ++i) {
            c[i][0] = 1;
            for (int j = 1; j <= i; ++j) c[i][j] = c[i - 1][j - 1] + (j <= i - 1 ? c[i - 1][j] : 0u);
        }
    }
};
constexpr ClusterBinomials kClBinomialsHost = ClusterBinomials();
__constant__ ClusterBinomials kClBinomials = ClusterBinomials();

// also gives the set's first row (cluster_first_row), gathered on the way: members come out highest first
template <typename Table>
__device__ __forceinline__ uint32_t cluster_set_at(const Table& choose, uint32_t index, int size, int n, uint32_t& first_row) {
    uint32_t set = 0, rows = 0, above = 0;
    int b = n;
    for (int i = size; i >= 1; --i) {
        do { --b; } while (choose[b][i] > index);
        set |= 1u << b;
        index -= choose[b][i];
        rows += (above << b) + (((uint32_t)b << b) >> 1);
        ++above;
    }
    first_row = rows;
    return set;
}

// LDS of the level kernel: the image (quotient rows; lanes beyond a row read on into the next one, or into the queries
// after the last, and drop what they read; then the window queries), and the run minima of each wave.
struct ClusterLds {
    uint32_t query_off, run_off, total;
    int waves;
    __host__ __device__ static ClusterLds make(const ClusterLayout& y, int waves) {
        ClusterLds s;
        s.waves = waves;
        s.query_off = (uint32_t)y.q_image_bytes();
        s.run_off = s.query_off + (uint32_t)y.query_bytes();
        s.total = s.run_off + (uint32_t)(waves * cluster_run_dwords(cluster_mode(y.L))) * 4u;
        return s;
    }
    // as many waves on a compute unit as its 160 KB of LDS allow (a row is a chain of dependent steps, so what
    // counts is the number of rows in flight): two workgroups of 16, 12 or 8 if they fit, else one of 16
    __host__ static ClusterLds choose(const ClusterLayout& y) {
        for (int waves = 16; waves >= 8; waves -= 4) {
            const ClusterLds s = make(y, waves);
            if (2u * s.total <= 160u * 1024u) return s;
        }
        return make(y, 16);
    }
};

__device__ __forceinline__ uint32_t cl_pk_min3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

extern __shared__ __align__(16) unsigned char cl_smem[];   // of the level kernel

// the next larger set of as many nodes, and its first row
__device__ __forceinline__ uint32_t cluster_next_set(uint32_t set, uint32_t& first_row) {
    const uint32_t low = set & (0u - set), up = set + low;
    set = (((up ^ set) >> 2) >> (__ffs(set) - 1)) | up;
    uint32_t rows = 0, above = 0;
    for (uint32_t bits = set; bits; ++above) {
        const int b = 31 - __clz(bits);
        bits ^= 1u << b;
        rows += (above << b) + (((uint32_t)b << b) >> 1);
    }
    first_row = rows;
    return set;
}

// The same for an instance on fewer nodes and cuts: G sets to a wave, 64 / G lanes of two entries each, with every set's
// values in its lanes (C <= n - 1).  The parts of a wave take a run of consecutive sets each.  15 nodes of a paper-shaped
// cluster keep 11 to 18 of their 50 layers: eight sets to a wave up to 15 layers, six up to 19 (then five up to 23, four up to 31).
template <int C, int G>
__device__ __forceinline__ void cluster_level_parts(const ClusterLayout y, const uint32_t* query, uint32_t* run32, uint32_t* A32,
                                                    const uint32_t (*choose)[PPO_CLUSTER_MAX_N + 1], bool more, int run_top, int lane,
                                                    uint32_t wave_index, uint32_t total_waves) {
    constexpr int CA = C > 0 ? C : 1, kLanes = 64 / G, kRuns = G == 2 ? 6 : G < 8 ? 5 : 4;
    constexpr bool kRows16 = G == 4 || G == 8;   // a set's lanes lie in one row of 16
    const bool spare = lane >= G * kLanes;       // five and six sets leave four lanes
    const int part = spare ? G - 1 : lane / kLanes, hl = lane - part * kLanes, n = y.n, rd = y.rs / 2, L = y.L;
    const uint32_t inf2 = kClInf | (kClInf << 16), all = (1u << n) - 1u;
    const int e0 = 2 * hl, e1 = e0 + 1;
    const uint32_t end_keep = (e0 == L ? 0u : 0xFFFFu) | (e1 == L ? 0u : 0xFFFF0000u);   // rest[L] = 0
    const uint32_t end_set = (e0 == L ? kClZero : 0u) | (e1 == L ? kClZero << 16 : 0u);
    const uint32_t nsets = (uint32_t)__builtin_amdgcn_readfirstlane((int)choose[n][C]);
    const uint32_t per = (nsets + total_waves * (uint32_t)G - 1u) / (total_waves * (uint32_t)G);
    const uint32_t u = (wave_index * (uint32_t)G + (uint32_t)part) * per;
    const uint32_t u_end = spare ? u : u + per < nsets ? u + per : nsets;
    uint32_t mp = (1u << C) - 1u, first_row = 0;
    if (u < u_end) mp = cluster_set_at(choose, u, C, n, first_row);
    const unsigned char* runb = reinterpret_cast<const unsigned char*>(run32) + part * (kLanes * 4);
    const uint32_t q_node = (uint32_t)(rd * 4);
    for (uint32_t it = 0; it < per; ++it) {
        const bool mine = u + it < u_end;
        if (__ballot(mine) == 0ull) break;
        uint32_t a[CA], moff[CA];
        {
            const uint32_t* arow = A32 + first_row * (uint32_t)rd + (uint32_t)hl;
            uint32_t bits = mp;
#pragma unroll
            for (int m = 0; m < C; ++m) {
                moff[m] = __umul24((uint32_t)__builtin_ctz(bits), q_node) + (uint32_t)hl * 4u;
                bits &= bits - 1u;
                a[m] = (more && hl < rd) ? arow[m * rd] : inf2;
            }
        }
        uint32_t jb = all & ~mp;
        for (int left = n - C; left > 0; --left) {
            const uint32_t j = (uint32_t)__builtin_ctz(jb);
            jb &= jb - 1u;
            const uint2 qd = *reinterpret_cast<const uint2*>(query + j * 64u + e0);
            uint32_t v = inf2;
            if (more) {
                const uint32_t qj = __umul24(j, (uint32_t)n * q_node);
                uint32_t x[CA];
#pragma unroll
                for (int m = 0; m < C; ++m) x[m] = cl_pk_max(*reinterpret_cast<const uint32_t*>(cl_smem + qj + moff[m]), a[m]);
#pragma unroll
                for (int m = 0; m + 1 < C; m += 2) v = cl_pk_min3(v, x[m], x[m + 1]);
                if (C & 1) v = cl_pk_min(v, x[C - 1]);
            }
            v = (v & end_keep) | end_set;
            // minima over runs (see cluster_level_kernel); four and eight sets: shifts within 16 lanes
            run32[lane] = v;
            constexpr int kUp1 = kRows16 ? 0x101 : 0x130;
            const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kUp1, 0xF, 0xF, true);
            uint32_t cur = cl_pk_min(v, (v >> 16) | (next << 16));
            run32[64 + lane] = cur;
            cur = cl_pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, kUp1, 0xF, 0xF, true));
            run32[128 + lane] = cur;
            if (kRows16) {
                cur = cl_pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x102, 0xF, 0xF, true));
                run32[192 + lane] = cur;
                if (G == 4) {
                    cur = cl_pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x104, 0xF, 0xF, true));
                    run32[256 + lane] = cur;
                }
            } else {
                const uint32_t up1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x130, 0xF, 0xF, true);
                cur = cl_pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)up1, 0x130, 0xF, 0xF, true));
                run32[192 + lane] = cur;
#pragma unroll
                for (int r = 4; r < kRuns; ++r) {
                    if (r > run_top) break;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    cur = cl_pk_min(cur, run32[(r - 1) * 64 + ((lane + (1 << (r - 2))) & 63)]);
                    run32[r * 64 + lane] = cur;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const uint32_t r1 = *reinterpret_cast<const uint16_t*>(runb + (qd.x & 0xFFFFu)) | (uint32_t)*reinterpret_cast<const uint16_t*>(runb + (qd.y & 0xFFFFu)) << 16;
            const uint32_t r2 = *reinterpret_cast<const uint16_t*>(runb + (qd.x >> 16)) | (uint32_t)*reinterpret_cast<const uint16_t*>(runb + (qd.y >> 16)) << 16;
            // row of j within R' + j: see cluster_level_kernel
            const uint32_t below = mp & ((1u << j) - 1u), above = (uint32_t)__popc((mp >> j) >> 1);
            const uint32_t row = first_row + (above << j) + ((j << j) >> 1) + below + (uint32_t)__popc(below);
            if (hl < rd && mine) A32[row * (uint32_t)rd + (uint32_t)hl] = cl_pk_min(r1, r2);
            __builtin_amdgcn_wave_barrier();
        }
        if (C > 0 && u + it + 1u < u_end) mp = cluster_next_set(mp, first_row);
    }
}

// C = |R'| = level - 1: the rows of the set's members sit in C registers, in the order of the members
template <int C, int MODE>
__global__ __launch_bounds__(1024, 8) void cluster_level_kernel(ClusterLayout y,
                                                                const unsigned char* __restrict__ ws,
                                                                uint16_t* __restrict__ rows, int pmax) {
    constexpr int level = C + 1, CA = C > 0 ? C : 1, G = cluster_sets_per_wave(MODE), kLanes = 64 / G;
    constexpr int kPitch = cluster_run_pitch(MODE), kRuns = cluster_run_levels(MODE);
    const int L = y.L, n = y.n, rd = y.rs / 2;
    const int inst = blockIdx.y, tid = threadIdx.x, lane = tid & 63, hl = lane & (kLanes - 1);
    const bool second = G == 2 && lane >= kLanes;   // lanes of the second set
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // the same in all lanes: keeps the set in scalar registers
    const int threads = blockDim.x, waves = threads >> 6;
    const ClusterLds lds = ClusterLds::make(y, waves);
    const unsigned char* base = ws + (size_t)inst * y.stride;
    const uint32_t* query = reinterpret_cast<const uint32_t*>(cl_smem + lds.query_off);
    uint32_t* run32 = reinterpret_cast<uint32_t*>(cl_smem + lds.run_off) + wave * cluster_run_dwords(MODE);
    uint32_t* A32 = reinterpret_cast<uint32_t*>(rows) + (size_t)inst * (y.rows_per_instance() * rd);
    if (cluster_flag(y, base)) {
        const ClusterLayout part = cluster_part_layout(y, base);
        if (C >= part.n) return;
        // as many waves as have a set to work on
        // entries 0 .. L of a set in its lanes
        const uint32_t G = part.L <= 15 ? 8u : part.L <= 19 ? 6u : part.L <= 23 ? 5u : part.L <= 31 ? 4u : 2u, nsets = kClBinomials.c[part.n][C];
        if (blockIdx.x * (uint32_t)waves * G >= nsets) return;
        const ClusterLds small = ClusterLds::make(part, waves);
        const uint4* img = reinterpret_cast<const uint4*>(base + part.img_off);
        for (int i = tid; i < (int)(small.run_off / 16u); i += threads) reinterpret_cast<uint4*>(cl_smem)[i] = img[i];
        const int top = (int)*reinterpret_cast<const uint32_t*>(base + part.img_off + small.run_off);
        // a set from its index is a chain of look-ups: the coefficients lie in LDS (read from memory they were half of a level)
        uint32_t* choose = reinterpret_cast<uint32_t*>(cl_smem + small.run_off);
        for (int i = tid; i < (int)(kClBinomialBytes / 4u); i += threads) choose[i] = kClBinomials.c[0][i];
        uint32_t* run = reinterpret_cast<uint32_t*>(cl_smem + small.run_off + kClBinomialBytes) + wave * cluster_run_dwords(kClTwoSets);
        if (cluster_part_none(part.L) + lane < cluster_run_dwords(kClTwoSets)) run[cluster_part_none(part.L) + lane] = kClInf | (kClInf << 16);   // empty windows
        __syncthreads();
        const uint32_t* windows = reinterpret_cast<const uint32_t*>(cl_smem + small.query_off);
        const uint32_t index = blockIdx.x * (uint32_t)waves + (uint32_t)wave, total = gridDim.x * (uint32_t)waves;
        const bool goes_on = part.n - level + 1 < pmax;
        const auto coefficients = reinterpret_cast<const uint32_t(*)[PPO_CLUSTER_MAX_N + 1]>(choose);
        if (G == 8u) cluster_level_parts<C, 8>(part, windows, run, A32, coefficients, goes_on, top, lane, index, total);
        else if (G == 6u) cluster_level_parts<C, 6>(part, windows, run, A32, coefficients, goes_on, top, lane, index, total);
        else if (G == 5u) cluster_level_parts<C, 5>(part, windows, run, A32, coefficients, goes_on, top, lane, index, total);
        else if (G == 4u) cluster_level_parts<C, 4>(part, windows, run, A32, coefficients, goes_on, top, lane, index, total);
        else cluster_level_parts<C, 2>(part, windows, run, A32, coefficients, goes_on, top, lane, index, total);
        return;
    }
    const bool more = n - level + 1 < pmax;   // segments up to and including this row's: n - level + 1
    // quotient rows and window queries: a straight copy of the image the tables kernels left (16 bytes a thread)
    {
        const uint4* img = reinterpret_cast<const uint4*>(base + y.img_off);
        uint4* dst = reinterpret_cast<uint4*>(cl_smem);
        const int first = more ? 0 : (int)(lds.query_off / 16u), count = (int)(lds.run_off / 16u);   // the quotient rows only if used
        for (int i = first + tid; i < count; i += threads) dst[i] = img[i];
    }
    const int run_top = (int)*reinterpret_cast<const uint32_t*>(base + y.img_off + lds.run_off);
    const uint32_t inf2 = kClInf | (kClInf << 16);
    // 128 layers: entry 128 of rest follows the lanes' in every run row, +inf after it; these never change
    const uint32_t after_last = kClZero | (kClInf << 16);
    if (MODE == kClWide)
        for (int i = lane; i < kRuns * (kPitch - 64); i += 64)
            run32[i / (kPitch - 64) * kPitch + 64 + i % (kPitch - 64)] = i % (kPitch - 64) ? inf2 : after_last;
    if (lane < cluster_run_dwords(MODE) - kRuns * kPitch) run32[kRuns * kPitch + lane] = inf2;
    __syncthreads();
    const uint32_t all = (1u << n) - 1u;
    const int e0 = 2 * hl, e1 = e0 + 1;
    // rest[L] = 0: the half of entry L is cleared and set to the code of 0
    const uint32_t end_keep = (e0 == L ? 0u : 0xFFFFu) | (e1 == L ? 0u : 0xFFFF0000u);
    const uint32_t end_set = (e0 == L ? kClZero : 0u) | (e1 == L ? kClZero << 16 : 0u);
    // A wave takes a run of consecutive sets: the first from its index (binomial table, a chain of dependent
    // scalar loads), each further one from the one before (the next larger number with as many bits set).
    const uint32_t nsets = kClBinomials.c[n][C];
    const uint32_t total_waves = gridDim.x * waves;
    const uint32_t per_wave = ((nsets + total_waves - 1u) / total_waves + (uint32_t)G - 1u) / (uint32_t)G * (uint32_t)G;
    uint32_t u = (blockIdx.x * waves + wave) * per_wave;
    const uint32_t u_end = u + per_wave < nsets ? u + per_wave : nsets;
    uint32_t mp = 0, first_row = 0;
    if (u < u_end) mp = cluster_set_at(kClBinomials.c, u, C, n, first_row);
    for (; u < u_end; u += (uint32_t)G) {
        const bool pair = G == 2 && u + 1u < u_end;
        uint32_t mp2 = mp, first_row2 = first_row;
        if (C > 0 && pair) mp2 = cluster_next_set(mp, first_row2);
        uint32_t a[CA];      // row A[R'][member m], two entries per lane
        int moff[CA];        // where member m's quotient rows are: of (j, m) from those of j (bytes)
        int mbelow[CA];      // one set to a wave: of (m, j) from those of j, if j < m (bytes)
        {
            const uint32_t mine = second ? first_row2 : first_row;
            const uint32_t* arow = A32 + (size_t)(mine * (uint32_t)rd) + hl;   // 32 bits hold an instance's dwords
            uint32_t bits = mp, bits2 = mp2;
#pragma unroll
            for (int m = 0; m < C; ++m) {
                const int b = __builtin_ctz(bits);
                bits &= bits - 1u;
                if (G == 2) {
                    const int b2 = __builtin_ctz(bits2);
                    bits2 &= bits2 - 1u;
                    moff[m] = ((second ? b2 : b) * rd + hl) * 4;
                } else {
                    // held as they are: products put off into the loop below made its scalar instructions the limit
                    // (level 11 of 20 nodes: 409 us)
                    moff[m] = __builtin_amdgcn_readfirstlane(b * (rd * 4));
                    mbelow[m] = __builtin_amdgcn_readfirstlane(ClusterLayout::below(b) * (rd * 4));
                }
                a[m] = (more && hl < rd) ? arow[m * rd] : inf2;
            }
        }
        // Where the rows of this set go: lane j works out the dword offset of row A[R' + j][j], once per set, and
        // the loop below picks it with a lane read instead of a dozen scalar instructions per row.  The first row
        // of R' + j from the first row of R' (j not in R'): the sets counted gain j's own term, and every member of
        // R' below j has one more member above it (their terms grow by 2^b each: `below` in all); then j's place
        // among the members.
        uint32_t out_off;
        {
            const uint32_t jl = (uint32_t)lane & 31u, set = second ? mp2 : mp;
            const uint32_t below = set & ((1u << jl) - 1u);
            const uint32_t above = (uint32_t)__popc((set >> jl) >> 1);
            out_off = ((second ? first_row2 : first_row) + (above << jl) + ((jl << jl) >> 1) + below + (uint32_t)__popc(below)) * (uint32_t)rd;
        }
        uint32_t jb = all & ~mp, jb2 = all & ~mp2;
        for (int left = n - C; left > 0; --left) {
            const int j = __builtin_ctz(jb), j2 = __builtin_ctz(jb2);
            jb &= jb - 1u;
            jb2 &= jb2 - 1u;
            const int my_j = second ? j2 : j;
            const uint2 qd = *reinterpret_cast<const uint2*>(query + my_j * (2 * kLanes) + e0);
            uint32_t v = inf2;
            if (more) {
                uint32_t x[CA];
                if (G == 2) {
                    const unsigned char* qj = cl_smem + my_j * (n * rd * 4);
#pragma unroll
                    for (int m = 0; m < C; ++m) x[m] = cl_pk_max(*reinterpret_cast<const uint32_t*>(qj + moff[m]), a[m]);
                } else {
                    const int joff = __builtin_amdgcn_readfirstlane(j * (rd * 4));
                    const int jbelow = __builtin_amdgcn_readfirstlane(ClusterLayout::below(j) * (rd * 4));
#pragma unroll
                    for (int m = 0; m < C; ++m) {
                        const int r1 = jbelow + moff[m], r2 = mbelow[m] + joff;
                        x[m] = cl_pk_max(*reinterpret_cast<const uint32_t*>(cl_smem + lane * 4 + (r1 > r2 ? r1 : r2)), a[m]);
                    }
                }
#pragma unroll
                for (int m = 0; m + 1 < C; m += 2) v = cl_pk_min3(v, x[m], x[m + 1]);
                if (C & 1) v = cl_pk_min(v, x[C - 1]);
            }
            v = (v & end_keep) | end_set;
            // minima over runs of 2^r entries starting at each entry; a run that passes the end of the row holds
            // whatever lies there and is never asked for (wave shift left by one: lane i reads lane i + 1; the last
            // lane of a row of 128 gets the entries after it)
            auto up_one = [&](uint32_t x, uint32_t after) -> uint32_t {
                return MODE == kClWide ? (uint32_t)__builtin_amdgcn_update_dpp((int)after, (int)x, 0x130, 0xF, 0xF, false)
                                       : (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x130, 0xF, 0xF, true);
            };
            run32[lane] = v;
            const uint32_t next = up_one(v, after_last);
            uint32_t cur = cl_pk_min(v, (v >> 16) | (next << 16));
            run32[kPitch + lane] = cur;
            cur = cl_pk_min(cur, up_one(cur, after_last));
            run32[2 * kPitch + lane] = cur;
            cur = cl_pk_min(cur, up_one(up_one(cur, after_last), inf2));
            run32[3 * kPitch + lane] = cur;
#pragma unroll
            for (int r = 4; r < kRuns; ++r) {
                if (r > run_top) break;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                cur = cl_pk_min(cur, run32[(r - 1) * kPitch + lane + (1 << (r - 2))]);
                run32[r * kPitch + lane] = cur;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const unsigned char* runb = reinterpret_cast<const unsigned char*>(run32) + (second ? kLanes * 4 : 0);
            uint32_t res[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t d = h ? qd.y : qd.x;
                const uint32_t r1 = *reinterpret_cast<const uint16_t*>(runb + (d & 0xFFFFu));
                const uint32_t r2 = *reinterpret_cast<const uint16_t*>(runb + (d >> 16));
                res[h] = r1 < r2 ? r1 : r2;
            }
            // row of j within R' + j: after the members below it
            uint32_t row_off = (uint32_t)__builtin_amdgcn_readlane((int)out_off, j);
            if (G == 2) {
                const uint32_t row_off2 = (uint32_t)__builtin_amdgcn_readlane((int)out_off, kLanes + j2);
                row_off = second ? row_off2 : row_off;
            }
            if (hl < rd && (!second || pair)) A32[(size_t)row_off + hl] = res[0] | (res[1] << 16);
            __builtin_amdgcn_wave_barrier();
        }
        if (C > 0 && u + (uint32_t)G < u_end) {
            first_row = first_row2;
            mp = cluster_next_set(mp2, first_row);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The optimum, the smallest optimal sequence and its cuts: one workgroup per instance.  With beta* known
// (the least A[All][j][0]) every further question is a yes or no, "can this be done with all links at most
// beta*", so the walk keeps sets of cuts as bit masks: F = cuts that the chosen prefix reaches (all its links
// at most beta*), G_j = those of F whose link into candidate j is at most beta*.  Candidate j at a position
// completes to an optimum iff A[unused][j][e] <= beta* for some e in G_j (one row of A, one wave per
// candidate); the smallest such node is taken, and F for the next position is the set of cuts that a window
// of that node starting in G_j covers.  hi[j][.] does not decrease, so the latest start below a cut decides.
// ---------------------------------------------------------------------------------------------
constexpr int kClTraceWaves = 16;   // at most; a launch uses min(n, 16) waves per workgroup

__global__ __launch_bounds__(kClTraceWaves * 64) void cluster_trace_kernel(ClusterLayout whole,
                                                                          const unsigned char* __restrict__ ws,
                                                                          const uint16_t* __restrict__ rows, int pmax,
                                                                          float* __restrict__ beta_out,
                                                                          int32_t* __restrict__ segs_out,
                                                                          int32_t* __restrict__ cuts_out,
                                                                          int32_t* __restrict__ order_out) {
    __shared__ unsigned char hi_s[PPO_CLUSTER_MAX_N * (PPO_MAX_L + 1)];
    __shared__ unsigned long long cand_s[PPO_CLUSTER_MAX_N][2];    // G_j of every candidate of this position
    __shared__ unsigned long long start_s[PPO_CLUSTER_MAX_N][2];   // G of the node chosen at every position
    __shared__ uint32_t ok_s[PPO_CLUSTER_MAX_N];
    __shared__ int seq[PPO_CLUSTER_MAX_N];
    const int inst = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned char* base = ws + (size_t)inst * whole.stride;
    const ClusterLayout y = cluster_layout(whole, base);
    const int L = y.L, n = y.n;
    const uint16_t* __restrict__ qc = reinterpret_cast<const uint16_t*>(base + y.qc_off);
    const float* __restrict__ dec = reinterpret_cast<const float*>(base + y.dec_off);
    const uint16_t* A = rows + (size_t)inst * (whole.rows_per_instance() * whole.rs);
    __shared__ unsigned char cut_s[PPO_MAX_L + 1], node_s[PPO_CLUSTER_MAX_N];   // the whole instance's
    if (cluster_reduced(whole, base)) {
        const ClusterRecord r = *reinterpret_cast<const ClusterRecord*>(base + whole.record_off());
        for (int e = tid; e < 128; e += (int)blockDim.x)
            if ((r.cuts[e >> 6] >> (e & 63)) & 1ull)
                cut_s[1 + (e >= 64 ? __popcll(r.cuts[0]) : 0) + __popcll(r.cuts[e >> 6] & ((1ull << (e & 63)) - 1ull))] = (unsigned char)e;
        for (int j = tid; j < whole.n; j += (int)blockDim.x)
            if ((r.nodes >> j) & 1u) node_s[__popc(r.nodes & ((1u << j) - 1u))] = (unsigned char)j;
    } else {
        for (int e = tid; e <= L; e += (int)blockDim.x) cut_s[e] = (unsigned char)e;
        for (int j = tid; j < n; j += (int)blockDim.x) node_s[j] = (unsigned char)j;
    }
    float* beta = beta_out + inst;
    int32_t* order = order_out + (size_t)inst * whole.n;
    int32_t* cuts = cuts_out ? cuts_out + (size_t)inst * (whole.n - 1) : nullptr;
    const int threads = blockDim.x, waves = threads >> 6;
    for (int i = tid; i < n * (L + 1); i += threads) hi_s[i] = base[y.hi_off + i];
    for (int i = tid; i < whole.n; i += threads) order[i] = -1;
    if (cuts)
        for (int i = tid; i < whole.n - 1; i += threads) cuts[i] = -1;
    __syncthreads();
    auto wave_min = [&](uint32_t v) -> uint32_t {
        for (int off = 32; off >= 1; off >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)v, off, 64);
            v = o < v ? o : v;
        }
        return v;
    };
    auto hi = [&](int j, int e) -> int { return hi_s[j * (L + 1) + e]; };
    const uint32_t all = (1u << n) - 1u;
    // every wave takes the minimum itself: the same value in all of them
    const uint32_t best = wave_min(lane < n ? (uint32_t)A[((size_t)cluster_first_row(all, n) + lane) * y.rs] : kClInf);
    if (best >= kClInf) {
        if (tid == 0) {
            *beta = __uint_as_float(kInfBits);
            segs_out[inst] = 0;
        }
        return;
    }
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
    unsigned long long F0 = 1ull, F1 = 0ull;   // the first segment starts at 0
    uint32_t used = 0;
    int last = -1, p = 0;
    for (int s = 0; s < pmax; ++s) {
        const uint32_t unused = all & ~used;
        const uint32_t first_row = cluster_first_row(unused, n);
        for (int j = wave; j < n; j += waves) {
            if ((used >> j) & 1u) {
                if (lane == 0) ok_s[j] = 0u;
                continue;
            }
            const uint16_t* __restrict__ a = A + (size_t)(first_row + (uint32_t)__popc(unused & ((1u << j) - 1u))) * y.rs;
            const uint16_t* __restrict__ q = qc + (s ? pair_index(last, j, n) * L : 0);
            unsigned long long g[2], ok[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int e = lane + 64 * h;
                // both requested before either is waited for
                const uint32_t link = q[e >= 1 && e < L ? e - 1 : 0], row = a[e < L ? e : 0];
                const bool in_f = (((h ? F1 : F0) >> lane) & 1ull) && e < L;
                const bool in_g = in_f && (s == 0 || link <= best);   // beyond the first position F holds no cut 0
                g[h] = __ballot(in_g);
                ok[h] = __ballot(in_g && row <= best);
            }
            if (lane == 0) {
                cand_s[j][0] = g[0];
                cand_s[j][1] = g[1];
                ok_s[j] = (ok[0] | ok[1]) != 0ull ? 1u : 0u;
            }
        }
        __syncthreads();
        const unsigned long long ok = __ballot(lane < n && ok_s[lane < n ? lane : 0] != 0u);
        const int chosen = ok ? __ffsll((long long)ok) - 1 : -1;
        if (chosen < 0) break;   // cannot happen: some completion of the prefix reaches `best`
        const unsigned long long G0 = cand_s[chosen][0], G1 = cand_s[chosen][1];
        if (tid == 0) {
            seq[s] = chosen;
            start_s[s][0] = G0;
            start_s[s][1] = G1;
        }
        // the prefix itself is optimal: it sorts before its extensions
        const bool complete = covered(G0, G1, chosen, L);
        F0 = __ballot(lane >= 1 && lane < L && covered(G0, G1, chosen, lane));
        F1 = __ballot(lane + 64 < L && covered(G0, G1, chosen, lane + 64));
        __syncthreads();
        used |= 1u << chosen;
        last = chosen;
        p = s + 1;
        if (complete) break;
    }
    if (wave != 0) return;
    // cuts: latest segment first, each time the smallest start (reached by the prefix, link at most beta*)
    // whose window covers the end
    int e = L;
    for (int s = p - 1; s >= 1 && cuts; --s) {
        const int js = seq[s];
        const unsigned long long m0 = __ballot(((start_s[s][0] >> lane) & 1ull) && lane < e && hi(js, lane) >= e);
        const unsigned long long m1 =
            __ballot(((start_s[s][1] >> lane) & 1ull) && lane + 64 < e && hi(js, lane + 64 < L ? lane + 64 : L) >= e);
        if (!(m0 | m1)) break;   // cannot happen: e was reached from such a start
        const int first = m0 ? __ffsll((long long)m0) - 1 : 63 + __ffsll((long long)m1);
        if (lane == 0) cuts[s - 1] = (int32_t)cut_s[first];
        e = first;
    }
    if (lane == 0) {
        *beta = dec[best - kClZero];
        segs_out[inst] = p;
        for (int s = 0; s < p; ++s) order[s] = node_s[seq[s]];
    }
}

// The image of the level kernel's LDS tables (needs hi and the codes): one workgroup per instance.
//   quotient rows: entry e of the row of (j, j''): q_{j,j''}[e-1] for 1 <= e <= L-1 (the cuts with a link), else +inf;
//   window queries: the window (e, hi[j][e]] of node j at entry e is covered by two runs of 2^k entries, k the
//   largest with 2^k <= its length: the one starting at e + 1 and the one ending at hi.  The table holds the byte
//   offsets of their minima within a wave's run minima, 16 bits each; no window: twice an entry that is +inf;
//   last, the largest k.
__global__ __launch_bounds__(kClPreThreads) void cluster_image_kernel(ClusterLayout whole, unsigned char* __restrict__ ws) {
    __shared__ int top_s;
    const int inst = blockIdx.x, tid = threadIdx.x;
    unsigned char* base = ws + (size_t)inst * whole.stride;
    const ClusterLayout y = cluster_layout(whole, base);
    const int L = y.L, n = y.n, mode = cluster_mode(L);
    const int pitch = cluster_run_pitch(mode), per_node = 128 / cluster_sets_per_wave(mode);
    const uint16_t* __restrict__ qc = reinterpret_cast<const uint16_t*>(base + y.qc_off);
    uint16_t* q16 = reinterpret_cast<uint16_t*>(base + y.img_off);
    uint32_t* query = reinterpret_cast<uint32_t*>(base + y.img_off + y.q_image_bytes());
    if (tid == 0) top_s = 0;
    __syncthreads();
    // a group of 64 threads per row
    const int nrows = mode == kClTwoSets ? n * n : y.npairs;
    for (int r = tid >> 6; r < nrows; r += kClPreThreads / 64) {
        int a, b;
        if (mode == kClTwoSets) {
            a = r / n;
            b = r - a * n;
        } else {
            b = 1;
            while (ClusterLayout::below(b + 1) <= r) ++b;
            a = r - ClusterLayout::below(b);
        }
        const uint16_t* __restrict__ q = qc + (a != b ? pair_index(a, b, n) : 0) * L;
        for (int e = tid & 63; e < y.rs; e += 64)
            q16[r * y.rs + e] = (uint16_t)((a != b && e >= 1 && e <= L - 1) ? q[e - 1] : kClInf);
    }
    for (int i = nrows * y.rs + tid; i < (int)(y.q_image_bytes() / 2); i += kClPreThreads) q16[i] = (uint16_t)kClInf;   // the padding
    const uint32_t none = (uint32_t)(cluster_reduced(whole, base) ? cluster_part_none(L) : cluster_run_levels(mode) * pitch) * 4u;
    int top_run = 0;
    for (int i = tid; i < n * per_node; i += kClPreThreads) {
        const int j = i / per_node, e = i - j * per_node;
        const int top = e < L ? (int)base[y.hi_off + j * (L + 1) + e] : 0;
        uint32_t o1 = none, o2 = none;
        if (top > e) {
            int k = 31 - __clz(top - e);
            k = k > cluster_run_levels(mode) - 1 ? cluster_run_levels(mode) - 1 : k;
            o1 = (uint32_t)(k * pitch * 4 + (e + 1) * 2);
            o2 = (uint32_t)(k * pitch * 4 + (top - (1 << k) + 1) * 2);
            top_run = k > top_run ? k : top_run;
        }
        query[i] = o1 | (o2 << 16);
    }
    // (one atomic a wave: an atomic by every thread made the table's kernel 8 us longer for 1024 instances of 12 layers)
    for (int off = 32; off >= 1; off >>= 1) {
        const int o = __shfl_xor(top_run, off, 64);
        top_run = o > top_run ? o : top_run;
    }
    if ((tid & 63) == 0) atomicMax(&top_s, top_run);
    __syncthreads();
    if (tid == 0) query[n * per_node] = (uint32_t)top_s;
}

// Whether a search is confined to the nodes and cuts that can matter (ppo_cluster_bound.hip).  That costs about 45 us before
// the levels, 10 to 15 where nine nodes do not hold the chain, and may leave little out: paper-shaped clusters of 16 MB devices
// keep all their nodes.  Measured in us, without and with it: one cluster of 16 such nodes 239 / 234, 16 of 13 nodes 236 / 224, 128
// of 11 nodes 277 / 229, but 128 of 10 nodes 177 / 185, 16 of 12 nodes 162 / 187, one of 14 nodes 176 / 193.  Mixed
// capacities, 100 layers: one of 20 nodes 2040 / 120 to 320, one of 16 nodes 275 to 309 / 95 to 178, 128 of 11 nodes 418 / 218; 20 layers: 64 of
// 13 nodes 390 / 238, but 132 of 12 nodes 447 / 500 and 288 of 11 nodes 455 / 541 (26 layers: 474 / 250 and 478 / 367).  Nothing to
// leave out: short of memory on the nine nodes, 16 nodes and 100 layers 252 / 271, 288 of 11 nodes 795 / 827; one transfer size
// and bandwidth, 16 nodes and 50 layers 223 / 262, 64 of 13 nodes 463 / 500.  With fewer segments allowed than nodes the upper
// levels are not searched, and those that are start from the nodes' number, which the host would not know.
static bool cluster_may_be_confined(int L, int n, int pmax) { return pmax == n && n >= (L >= 24 ? 11 : 13); }
static bool cluster_confined(int L, int n, int n_inst, int pmax) {
    return cluster_may_be_confined(L, n, pmax) && (n >= 16 || ((unsigned long long)n_inst * (unsigned long long)n << (n - 1)) >= 800000ull);
}

hipError_t launch_cluster_tables(const float* t, const float* m, const float* M, const float* B, int L, int n,
                                 int n_inst, int pmax, void* ws, hipStream_t stream) {
    const ClusterLayout y = ClusterLayout::make(L, n, cluster_confined(L, n, n_inst, pmax));
    unsigned char* w = static_cast<unsigned char*>(ws);
    hipError_t e;
    if (y.may_be_reduced) {
        e = launch_cluster_reduce(t, m, M, B, y, n_inst, w, stream);
    } else {
        hipLaunchKernelGGL(cluster_tables_kernel, dim3(n_inst), dim3(kClPreThreads), 0, stream, t, m, M, B, y, w);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    if (y.nq > 0) {
        const int slices = (y.nq + kClCountSlice - 1) / kClCountSlice;
        const uint32_t lds_bytes = ((uint32_t)y.nq + (uint32_t)kClCountSlice) * 4u;
        static std::atomic<uint64_t> lds_allowed{0};
        e = allow_full_lds(reinterpret_cast<const void*>(&cluster_count_kernel), lds_allowed);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(cluster_count_kernel, dim3(slices, n_inst), dim3(kClCountThreads), lds_bytes, stream, y, w);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(cluster_image_kernel, dim3(n_inst), dim3(kClPreThreads), 0, stream, y, w);
    return hipGetLastError();
}

// rows of `n_inst` instances (tables at ws, rows at `rows`), levels n - pmax + 1 .. n, then the trace
// one instantiation of the level kernel per set size
using ClLevelLaunch = hipError_t (*)(dim3, dim3, uint32_t, hipStream_t, const ClusterLayout&, const unsigned char*,
                                     uint16_t*, int);
template <int C, int MODE>
static hipError_t cluster_launch_mode(dim3 grid, dim3 block, uint32_t lds_bytes, hipStream_t stream, const ClusterLayout& y,
                                      const unsigned char* ws, uint16_t* rows, int pmax) {
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&cluster_level_kernel<C, MODE>), lds_allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((cluster_level_kernel<C, MODE>), grid, block, lds_bytes, stream, y, ws, rows, pmax);
    return hipGetLastError();
}
template <int C>
static hipError_t cluster_launch_level(dim3 grid, dim3 block, uint32_t lds_bytes, hipStream_t stream, const ClusterLayout& y,
                                       const unsigned char* ws, uint16_t* rows, int pmax) {
    const int mode = cluster_mode(y.L);
    return mode == kClTwoSets ? cluster_launch_mode<C, kClTwoSets>(grid, block, lds_bytes, stream, y, ws, rows, pmax)
           : mode == kClOneSet ? cluster_launch_mode<C, kClOneSet>(grid, block, lds_bytes, stream, y, ws, rows, pmax)
                               : cluster_launch_mode<C, kClWide>(grid, block, lds_bytes, stream, y, ws, rows, pmax);
}
template <int... Cs>
static constexpr std::array<ClLevelLaunch, sizeof...(Cs)> cluster_level_table(std::integer_sequence<int, Cs...>) {
    return {{&cluster_launch_level<Cs>...}};
}
static const std::array<ClLevelLaunch, PPO_CLUSTER_MAX_N> kClLevelLaunch =
    cluster_level_table(std::make_integer_sequence<int, PPO_CLUSTER_MAX_N>{});

hipError_t launch_cluster_solve(int L, int n, int n_inst, int pmax, const void* ws, void* rows, float* beta_out,
                                int32_t* segs_out, int32_t* cuts_out, int32_t* order_out, hipStream_t stream) {
    // (the tables may have been made for more instances at once than are searched here: their flag says)
    const ClusterLayout y = ClusterLayout::make(L, n, cluster_may_be_confined(L, n, pmax));
    const unsigned char* w = static_cast<const unsigned char*>(ws);
    uint16_t* r = static_cast<uint16_t*>(rows);
    const ClusterLds lds = ClusterLds::choose(y);
    const uint32_t resident = 256u * (2u * lds.total <= 160u * 1024u ? 2u : 1u);   // workgroups the chip holds
    const uint32_t sets_each = (uint32_t)(lds.waves * cluster_sets_per_wave(cluster_mode(L)));
    hipError_t e = hipSuccess;
    for (int level = n - pmax + 1; level <= n; ++level) {
        // no more workgroups than stay resident (each stages the quotient table once)
        uint32_t blocks = (kClBinomialsHost.c[n][level - 1] + sets_each - 1u) / sets_each;
        const uint32_t cap = (resident + (uint32_t)n_inst - 1u) / (uint32_t)n_inst;
        if (blocks > cap) blocks = cap;
        e = kClLevelLaunch[level - 1](dim3(blocks, n_inst), dim3(lds.waves * 64), lds.total, stream, y, w, r, pmax);
        if (e != hipSuccess) return e;
    }
    const int trace_waves = n < kClTraceWaves ? n : kClTraceWaves;   // one wave per candidate node
    hipLaunchKernelGGL(cluster_trace_kernel, dim3(n_inst), dim3(trace_waves * 64), 0, stream, y, w, r, pmax,
                       beta_out, segs_out, cuts_out, order_out);
    return hipGetLastError();
}

}  // namespace ppo
