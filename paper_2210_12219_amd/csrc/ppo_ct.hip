// The search with the compute-time term of Sec. I, Eq. 1: beta is the largest stage of the pipeline, compute
// stages (work of a segment over the speed of its node) and communication stages (Eq. 3) alike.  The paper
// drops the compute stages (Eq. 2); this file keeps them.
//
//   comp(i, e, j) = (float)((Q[e] - Q[i]) / (double)v[j])     Q: binary64 prefix sums of the per-layer work
//   D_0[e] = comp(0, e, pi_0)                                  if layers [0, e) fit node pi_0
//   D_s[e] = min over i in [max(lo[pi_s][e], s), e-1] of max(D_{s-1}[i], q_{pi_{s-1},pi_s}[i-1], comp(i, e, pi_s))
//   beta(pi) = D_{k-1}[L]
//
// The compute stage depends on both ends of a segment, so there are about k L^2 / 2 distinct stage values per
// instance: too many for the 16-bit order codes of the search without the term.  This path therefore works on
// the binary32 values themselves (as unsigned bit patterns: they are non-negative).  The search goes over sets of
// nodes; single orderings (ppo_eval_orderings_ct) run one to a lane, the row in LDS, by the recurrence above.
#include "ppo_sets.h"

namespace ppo {

struct CtLayout {
    int L, k, npairs;
    uint32_t lo_off, q_off, ct_off, stride;   // bytes within one instance's slice
    __host__ __device__ static CtLayout make(int L, int k) {
        CtLayout y;
        y.L = L;
        y.k = k;
        y.npairs = k * (k - 1) / 2;
        size_t off = 0;
        y.lo_off = (uint32_t)off;                       // lo [k][L+1] u8: first legal segment start
        off = align_up(off + (size_t)k * (L + 1), 16);
        y.q_off = (uint32_t)off;                        // q [npairs][L] f32: t[i] / B[a][b], i < L-1
        off = align_up(off + (size_t)y.npairs * L * 4, 16);
        y.ct_off = (uint32_t)off;                       // ct [k][L+1][L+1] f32: comp(i, e, j) at [j][e][i], i < e
        off = align_up(off + (size_t)k * (L + 1) * (L + 1) * 4, 256);
        y.stride = (uint32_t)off;
        return y;
    }
};

size_t ct_tables_bytes(int L, int k) { return CtLayout::make(L, k).stride; }

constexpr int kCtPreThreads = 256;

__global__ __launch_bounds__(kCtPreThreads) void ct_tables_kernel(const float* __restrict__ t, const float* __restrict__ m,
                                                                  const float* __restrict__ w, const float* __restrict__ M,
                                                                  const float* __restrict__ v, const float* __restrict__ B,
                                                                  CtLayout y, unsigned char* __restrict__ ws) {
    __shared__ double P[PPO_MAX_L + 1], Q[PPO_MAX_L + 1];
    const int L = y.L, k = y.k, inst = blockIdx.x, tid = threadIdx.x, W = L + 1;
    const float* ti = t + (size_t)inst * L;
    const float* mi = m + (size_t)inst * L;
    const float* wi = w + (size_t)inst * L;
    const float* Mi = M + (size_t)inst * k;
    const float* vi = v + (size_t)inst * k;
    const float* Bi = B + (size_t)inst * k * k;
    unsigned char* base = ws + (size_t)inst * y.stride;
    if (tid == 0) {   // the definition fixes the order of the additions
        double a = 0.0, b = 0.0;
        P[0] = 0.0;
        Q[0] = 0.0;
        for (int i = 0; i < L; ++i) {
            a = a + (double)mi[i];
            b = b + (double)wi[i];
            P[i + 1] = a;
            Q[i + 1] = b;
        }
    }
    __syncthreads();
    unsigned char* lo = base + y.lo_off;
    for (int idx = tid; idx < k * W; idx += kCtPreThreads) {
        const int j = idx / W, e = idx - j * W;
        const double cap = (double)Mi[j];
        int i = 0;
        while (i < e && (P[e] - P[i]) > cap) ++i;
        lo[idx] = (unsigned char)i;
    }
    float* q = reinterpret_cast<float*>(base + y.q_off);
    for (int idx = tid; idx < y.npairs * L; idx += kCtPreThreads) {
        const int p = idx / L, i = idx - p * L;
        int a = 0, rem = p;
        while (rem >= k - 1 - a) { rem -= k - 1 - a; ++a; }
        const int b = a + 1 + rem;
        const float tv = ti[i] == 0.0f ? 0.0f : ti[i];   // a zero of either sign is +0
        q[idx] = i < L - 1 ? __fdiv_rn(tv, Bi[a * k + b]) : __uint_as_float(kInfBits);
    }
    float* ct = reinterpret_cast<float*>(base + y.ct_off);
    for (int idx = tid; idx < k * W * W; idx += kCtPreThreads) {
        const int j = idx / (W * W), rest = idx - j * W * W, e = rest / W, i = rest - e * W;
        ct[idx] = i < e ? __double2float_rn(__ddiv_rn(Q[e] - Q[i], (double)vi[j])) : __uint_as_float(kInfBits);
    }
}

// One DP of one ordering, in place in the lane's row (row[e * stride], binary32 bit patterns).
__device__ inline uint32_t ct_dp_one_ordering(uint64_t perm, int L, int k, const unsigned char* lo_s, const uint32_t* q_s,
                                              const uint32_t* __restrict__ ct, uint32_t* row, int stride) {
    const int W = L + 1;
    const int n0 = perm_at(perm, 0);
    const unsigned char* lo0 = lo_s + n0 * W;
    const uint32_t* ct0 = ct + (size_t)n0 * W * W;
    for (int e = 1; e <= L - (k - 1); ++e) row[e * stride] = lo0[e] == 0 ? ct0[e * W] : kInfBits;
    int prev = n0;
    for (int s = 1; s < k; ++s) {
        const int node = perm_at(perm, s);
        const uint32_t* q = q_s + pair_index(prev, node, k) * L;
        const unsigned char* lo = lo_s + node * W;
        const uint32_t* cj = ct + (size_t)node * W * W;
        for (int e = L - k + 1 + s; e >= s + 1; --e) {
            int first = lo[e];
            first = first > s ? first : s;
            uint32_t acc = kInfBits;
            const uint32_t* ce = cj + e * W;
            for (int i = first; i < e; ++i) {
                uint32_t c = row[i * stride];
                const uint32_t g = q[i - 1], h = ce[i];
                c = c > g ? c : g;
                c = c > h ? c : h;
                acc = c < acc ? c : acc;
            }
            row[e * stride] = acc;
        }
        prev = node;
    }
    return row[L * stride];
}

__global__ __launch_bounds__(256) void ct_enumerate_kernel(CtLayout y, const unsigned char* __restrict__ ws,
                                                          uint32_t rank_begin, uint32_t rank_end,
                                                          float* __restrict__ beta_export) {
    extern __shared__ __align__(16) unsigned char ct_smem[];
    const int L = y.L, k = y.k, inst = blockIdx.y, tid = threadIdx.x, T = blockDim.x;
    const unsigned char* base = ws + (size_t)inst * y.stride;
    // lo and q are contiguous at the start of the slice
    const uint32_t table_bytes = y.ct_off;
    for (uint32_t i = tid * 16u; i < table_bytes; i += (uint32_t)T * 16u)
        *reinterpret_cast<uint4*>(ct_smem + i) = *reinterpret_cast<const uint4*>(base + i);
    __syncthreads();
    const unsigned char* lo_s = ct_smem + y.lo_off;
    const uint32_t* q_s = reinterpret_cast<const uint32_t*>(ct_smem + y.q_off);
    const uint32_t* ct = reinterpret_cast<const uint32_t*>(base + y.ct_off);
    uint32_t* row = reinterpret_cast<uint32_t*>(ct_smem + table_bytes) + tid;
    const uint32_t span = rank_end - rank_begin;
    for (uint32_t off = blockIdx.x * (uint32_t)T + tid; off < span; off += gridDim.x * (uint32_t)T)
        beta_export[off] = __uint_as_float(ct_dp_one_ordering(unrank_packed(rank_begin + off, k), L, k, lo_s, q_s, ct, row, T));
}

// ---------------------------------------------------------------------------------------------
// The search: dynamic programming over the sets of nodes not yet used, as in ppo_subset.hip (recurrence, numbering of the
// rows, traceback), on binary32 patterns.  One workgroup per instance.  With the compute stage
//     A[{j}][j][e] = comp(e, L, j)                                                            if layers [e, L) fit node j
//     A[R][j][e]   = min over e' in (e, min(hi_j(e), L-1)] of max(rest[e'], comp(e, e', j)),   rest as in ppo_subset.hip
// comp does not decrease with e' (the weights of the work are >= 0 and both roundings are monotone), so rest may be
// replaced by its least value up to e': that one does not increase, and the minimum lies where the two cross.  The
// crossing is found by descending through minima over runs of 2^r entries: log2(window) steps instead of a candidate per
// entry of the window.  1024 x (50 layers, 6 nodes): 119 us, against 2.76 ms with a programme per ordering.
//
// What bounds it: the chain of dependent LDS reads of a row (six levels of runs, six steps of two reads each) with eight
// to twenty-four waves on a compute unit: of the time of the 3.7 waves on a SIMD 0.58 is spent waiting, 206 vector,
// 102 scalar and 37 LDS instructions a row fill 0.57, 0.28 and 0.26 of their units' time (1024 x (50, 6)).  The compute
// stages of an instance stay in LDS while two workgroups fit beside each other (a descent reads them once a step,
// scattered); beyond that, and for the rows, the caches hold them.
// ---------------------------------------------------------------------------------------------
namespace {

struct CtShared {
    uint32_t longest;
};
// H entries per lane: entry lane + 64 h
struct CtLds {
    uint32_t q_off, P_off, Q_off, t_off, hi_off, run_off, comp_off, total;
    __host__ __device__ static int run_levels(int H) { return H == 2 ? 7 : 6; }
    __host__ __device__ static uint32_t run_dwords(int H) { return (uint32_t)(run_levels(H) * 64 * H + 4); }
    __host__ __device__ static CtLds make(int L, int k, int H, int waves, bool comp_in_lds) {
        CtLds s;
        size_t off = 16;                                  // CtShared
        s.q_off = (uint32_t)off;                          // [k][k][64 H]: entry e of (j, j'') belongs to the cut e
        off += (size_t)k * k * 64 * H * 4;
        s.P_off = (uint32_t)off;
        off += (align_up((size_t)L, 64) + 2) * 8;
        s.Q_off = (uint32_t)off;
        off += (align_up((size_t)L, 64) + 2) * 8;
        s.t_off = (uint32_t)off;
        off += align_up((size_t)L, 4) * 4;
        s.hi_off = (uint32_t)off;
        off = align_up(off + (size_t)k * (L + 1), 16);
        s.run_off = (uint32_t)off;
        off += (size_t)waves * run_dwords(H) * 4;
        s.comp_off = (uint32_t)off;
        if (comp_in_lds) off += comp_count(L, k) * 4;
        s.total = (uint32_t)align_up(off, 16);
        return s;
    }
    // compute stages of an instance: comp(e, e', j) at [j][e][e' - e - 1]
    __host__ __device__ static size_t comp_count(int L, int k) { return (size_t)k * (size_t)(L * (L + 1) / 2); }
    __host__ __device__ static int comp_row(int L, int e) { return e * L - e * (e - 1) / 2; }
};

template <int C, int H>
__device__ __forceinline__ void ct_level(int k, int L, int lane, int wave, int waves, const uint32_t* q_s,
                                         const unsigned char* hi_s, uint32_t* run, const uint32_t* comp, uint32_t* rows,
                                         int run_top) {
    constexpr int kRow = 64 * H;
    const uint32_t all = (1u << k) - 1u, nsets = kSets.choose[k][C];
    const int T = L * (L + 1) / 2;
    int ec[H], crow[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        ec[h] = lane + 64 * h < L ? lane + 64 * h : L - 1;
        crow[h] = CtLds::comp_row(L, ec[h]) - 1;   // comp(e, e', j) at crow + j T + (e' - e)
    }
    for (uint32_t u = (uint32_t)wave; u < nsets; u += (uint32_t)waves) {
        const uint32_t entry = (uint32_t)__builtin_amdgcn_readfirstlane((int)kSets.order[kSets.first[C] + (int)u]);
        const uint32_t mp = entry & 0xFFFFu, first_row = entry >> 16;
        uint32_t a[C][H], qoff[C];
        {
            uint32_t bits = mp;
#pragma unroll
            for (int m = 0; m < C; ++m) {
                qoff[m] = (uint32_t)(__ffs(bits) - 1) * (uint32_t)(k * kRow) + (uint32_t)lane;
                bits &= bits - 1u;
#pragma unroll
                for (int h = 0; h < H; ++h) a[m][h] = rows[(first_row + m) * (uint32_t)L + (uint32_t)ec[h]];
            }
        }
        for (uint32_t jb = all & ~mp; jb; jb &= jb - 1u) {
            const int j = __ffs(jb) - 1;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                uint32_t v = kInfBits;
#pragma unroll
                for (int m = 0; m < C; ++m) {
                    const uint32_t g = q_s[qoff[m] + (uint32_t)(j * kRow + 64 * h)];
                    const uint32_t x = g > a[m][h] ? g : a[m][h];
                    v = x < v ? x : v;
                }
                run[lane + 64 * h] = v;
            }
            for (int r = 1; r <= run_top; ++r) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const uint32_t* below = run + (r - 1) * kRow + lane;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const uint32_t x = below[64 * h], y = below[64 * h + (1 << (r - 1))];
                    run[r * kRow + lane + 64 * h] = x < y ? x : y;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // the end of the longest stretch over which the least `rest` is still above the compute stage
            const uint32_t out = row_of(first_row, mp, (uint32_t)j) * (uint32_t)L;
            int hi[H], pos[H];
            uint32_t cur[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int top = hi_s[j * (L + 1) + ec[h]];
                hi[h] = top < L - 1 ? top : L - 1;
                pos[h] = ec[h];
                cur[h] = kInfBits;
            }
            for (int r = run_top; r >= 0; --r) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int end = pos[h] + (1 << r);
                    const int to = end <= hi[h] ? end : ec[h] + 1;   // beyond the window: any stage, not used
                    const uint32_t m = run[r * kRow + pos[h] + 1], stage = comp[crow[h] + j * T + (to - ec[h])];
                    const uint32_t least = m < cur[h] ? m : cur[h];
                    if (end <= hi[h] && least > stage) {
                        pos[h] = end;
                        cur[h] = least;
                    }
                }
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
                uint32_t res = cur[h];
                if (pos[h] < hi[h]) {   // the first end at which the stage is no longer below: nothing later is better
                    const uint32_t m = run[pos[h] + 1], stage = comp[crow[h] + j * T + (pos[h] + 1 - ec[h])];
                    const uint32_t least = m < cur[h] ? m : cur[h];
                    const uint32_t x = least > stage ? least : stage;
                    res = x < res ? x : res;
                }
                if (lane + 64 * h < L) rows[out + (uint32_t)(lane + 64 * h)] = res;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

}  // namespace

constexpr int kCtWaves = 8;

template <int H, bool LDSCOMP>
__global__ __launch_bounds__(kCtWaves * 64) void ct_solve_kernel(
    const float* __restrict__ t_in, const float* __restrict__ m_in, const float* __restrict__ w_in,
    const float* __restrict__ M_in, const float* __restrict__ v_in, const float* __restrict__ B_in, int L, int k, int n_inst,
    float* __restrict__ beta_out, int32_t* __restrict__ cuts_out, int32_t* __restrict__ order_out, uint32_t* slots,
    size_t slot_dwords) {
    extern __shared__ __align__(16) unsigned char ct_sm[];
    constexpr int threads = kCtWaves * 64, kRow = 64 * H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CtLds lds = CtLds::make(L, k, H, kCtWaves, LDSCOMP);
    CtShared& sh = *reinterpret_cast<CtShared*>(ct_sm);
    uint32_t* q_s = reinterpret_cast<uint32_t*>(ct_sm + lds.q_off);
    double* P = reinterpret_cast<double*>(ct_sm + lds.P_off);
    double* Q = reinterpret_cast<double*>(ct_sm + lds.Q_off);
    float* t_s = reinterpret_cast<float*>(ct_sm + lds.t_off);
    unsigned char* hi_s = ct_sm + lds.hi_off;
    uint32_t* run = reinterpret_cast<uint32_t*>(ct_sm + lds.run_off) + wave * CtLds::run_dwords(H);
    uint32_t* rows = slots + (size_t)blockIdx.x * slot_dwords;
    const uint32_t row_count = (uint32_t)k << (k - 1);
    uint32_t* comp = LDSCOMP ? reinterpret_cast<uint32_t*>(ct_sm + lds.comp_off) : rows + (size_t)row_count * L;
    const uint32_t all = (1u << k) - 1u;
    const int T = L * (L + 1) / 2;

    for (uint32_t inst = blockIdx.x; inst < (uint32_t)n_inst; inst += gridDim.x) {
        for (int i = tid; i < L; i += threads) {
            const float x = t_in[(size_t)inst * L + i];
            t_s[i] = x == 0.0f ? 0.0f : x;   // a zero of either sign is +0
        }
        if (tid == 0) sh.longest = 0u;
        if (wave < 2) {
            // prefix sums in index order in binary64: the weights by one wave, the work by another (all lanes of it add
            // and store the same)
            const float* src = (wave == 0 ? m_in : w_in) + (size_t)inst * L;
            double* dst = wave == 0 ? P : Q;
            double acc = 0.0;
            dst[0] = 0.0;
            for (int base = 0; base < L; base += 64) {
                const float x = base + lane < L ? src[base + lane] : 0.0f;
#pragma unroll
                for (int i = 0; i < 64; ++i) {
                    acc = acc + (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), i));
                    dst[base + i + 1] = acc;
                }
            }
        }
        __syncthreads();
        int longest = 0;
        for (int idx = tid; idx < k * (L + 1); idx += threads) {
            const int j = idx / (L + 1), e = idx - j * (L + 1);
            const double cap = (double)M_in[(size_t)inst * k + j], from = P[e];
            int good = e, step = 1;
            while (step < L) step <<= 1;
            for (; step >= 1; step >>= 1) {
                const int e2 = good + step;
                if (e2 <= L && P[e2] - from <= cap) good = e2;
            }
            hi_s[idx] = (unsigned char)good;
            if (good > e) {
                const int r = 31 - __clz(good - e);
                longest = r > longest ? r : longest;
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const int o = __shfl_xor(longest, off, 64);
            longest = o > longest ? o : longest;
        }
        if (lane == 0) atomicMax(&sh.longest, (uint32_t)longest);
        for (int idx = tid; idx < k * k * kRow; idx += threads) {
            const int e = idx & (kRow - 1), jj = idx / kRow, a = jj / k, b = jj - a * k;
            uint32_t c = kInfBits;
            if (a != b && e >= 1 && e <= L - 1)   // the element with the smaller row index is the one read
                c = __float_as_uint(__fdiv_rn(t_s[e - 1], B_in[(size_t)inst * k * k + (a < b ? jj : b * k + a)]));
            q_s[idx] = c < kInfBits ? c : kInfBits;
        }
        for (int idx = tid; idx < k * L * L; idx += threads) {
            const int j = idx / (L * L), rest = idx - j * L * L, e = rest / L, len = rest - e * L;   // e' = e + len + 1
            if (e + len < L) {
                const uint32_t c = __float_as_uint(
                    __double2float_rn(__ddiv_rn(Q[e + len + 1] - Q[e], (double)v_in[(size_t)inst * k + j])));
                comp[j * T + CtLds::comp_row(L, e) + len] = c < kInfBits ? c : kInfBits;
            }
        }
        __syncthreads();
        for (int idx = tid; idx < k * L; idx += threads) {   // sets of one node: its segment runs to the end of the chain
            const int j = idx / L, e = idx - j * L;
            rows[row_of(0u, 0u, (uint32_t)j) * (uint32_t)L + (uint32_t)e] =
                hi_s[j * (L + 1) + e] == L ? comp[j * T + CtLds::comp_row(L, e) + L - e - 1] : kInfBits;
        }
        __syncthreads();
        const int top = (int)sh.longest, run_top = top < CtLds::run_levels(H) - 1 ? top : CtLds::run_levels(H) - 1;
#define PPO_CT_LEVEL(C_)                                                                        \
    if (k > C_) {                                                                               \
        ct_level<C_, H>(k, L, lane, wave, kCtWaves, q_s, hi_s, run, comp, rows, run_top);       \
        __syncthreads();                                                                        \
    }
        PPO_CT_LEVEL(1)
        PPO_CT_LEVEL(2)
        PPO_CT_LEVEL(3)
        PPO_CT_LEVEL(4)
        PPO_CT_LEVEL(5)
        PPO_CT_LEVEL(6)
        PPO_CT_LEVEL(7)
        PPO_CT_LEVEL(8)
        PPO_CT_LEVEL(9)
        PPO_CT_LEVEL(10)
        PPO_CT_LEVEL(11)
#undef PPO_CT_LEVEL
        if (wave == 0) {
            // beta*, then the lexicographically smallest optimal ordering and its cuts (see ppo_subset.hip); the compute
            // stage shrinks with a later start, so the latest start below a cut decides here too
            uint32_t best = lane < k ? rows[(row_count - (uint32_t)k + (uint32_t)lane) * (uint32_t)L] : kInfBits;
            for (int off = 8; off >= 1; off >>= 1) {
                const uint32_t o = (uint32_t)__shfl_xor((int)best, off, 64);
                best = o < best ? o : best;
            }
            best = (uint32_t)__builtin_amdgcn_readfirstlane((int)best);
            int32_t* cuts = cuts_out + (size_t)inst * (k - 1);
            int32_t* order = order_out + (size_t)inst * k;
            if (lane == 0) beta_out[inst] = __uint_as_float(best);
            if (best >= kInfBits) {
                if (lane < k) order[lane] = -1;
                if (lane < k - 1) cuts[lane] = -1;
            } else {
                auto reaches = [&](int from, int to, int j) -> bool {   // 0 <= from < to <= L
                    return hi_s[j * (L + 1) + from] >= to && comp[j * T + CtLds::comp_row(L, from) + to - from - 1] <= best;
                };
                auto covered = [&](const unsigned long long* g, int j, int e2) -> bool {   // 1 <= e2 < L
                    unsigned long long m0 = g[0], m1 = 0;
                    if (e2 < 64)
                        m0 &= (1ull << e2) - 1ull;
                    else
                        m1 = g[1] & ((1ull << (e2 - 64)) - 1ull);
                    const int from = m1 ? 127 - __clzll((long long)m1) : m0 ? 63 - __clzll((long long)m0) : -1;
                    return from >= 0 && reaches(from, e2, j);
                };
                unsigned long long F[2] = {1ull, 0ull}, my_start[2] = {0ull, 0ull};
                uint32_t unused = all, first_row = row_count - (uint32_t)k;
                int last = 0, my_node = 0;
                for (int s = 0; s < k; ++s) {
                    int chosen = __ffs(unused) - 1;
                    unsigned long long Gc[2] = {0ull, 0ull};
                    for (uint32_t jb = unused; jb; jb &= jb - 1u) {
                        const int j = __ffs(jb) - 1;
                        const uint32_t* a = rows + (first_row + (uint32_t)__popc(unused & ((1u << j) - 1u))) * (uint32_t)L;
                        const uint32_t* q = q_s + (last * k + j) * kRow;
                        unsigned long long g[2] = {0ull, 0ull}, ok = 0ull;
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            const int e = lane + 64 * h;
                            const bool in_f = ((F[h] >> lane) & 1ull) && e < L;
                            const bool in_g = in_f && (s == 0 || q[e] <= best);   // beyond the first position F holds no cut 0
                            g[h] = __ballot(in_g);
                            ok |= __ballot(in_g && a[e] <= best);
                        }
                        if (ok) {
                            chosen = j;
                            Gc[0] = g[0];
                            Gc[1] = g[1];
                            break;
                        }
                    }
                    if (lane == s) {
                        my_node = chosen;
                        my_start[0] = Gc[0];
                        my_start[1] = Gc[1];
                    }
                    F[0] = __ballot(lane >= 1 && lane < L && covered(Gc, chosen, lane));
                    if (H == 2) F[1] = __ballot(lane + 64 < L && covered(Gc, chosen, lane + 64));
                    unused &= ~(1u << chosen);
                    first_row -= row_of(0u, unused, (uint32_t)chosen) - (uint32_t)__popc(unused & ((1u << chosen) - 1u));
                    last = chosen;
                }
                int e = L;
                for (int s = k - 1; s >= 1; --s) {
                    const int js = __builtin_amdgcn_readlane(my_node, s);
                    int first = -1;
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const unsigned long long start =
                            (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_start[h], s) |
                            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_start[h] >> 32), s) << 32);
                        const int i = lane + 64 * h;
                        const unsigned long long found = __ballot(((start >> lane) & 1ull) && i < e && reaches(i, e, js));
                        if (found && first < 0) first = 64 * h + __ffsll((long long)found) - 1;
                    }
                    if (lane == 0) cuts[s - 1] = first;
                    if (first < 0) break;   // cannot happen: e was reached from such a start
                    e = first;
                }
                if (lane < k) order[lane] = my_node;
            }
        }
        __syncthreads();   // the next instance overwrites what the last steps read
    }
}

static bool ct_comp_in_lds(int L, int k) {
    return 2u * CtLds::make(L, k, L <= 64 ? 1 : 2, kCtWaves, true).total <= (uint32_t)kLdsBytesPerCU;
}

// scratch of one workgroup: rows, then the compute stages if they are not in LDS
size_t ct_slot_bytes(int L, int k) {
    return align_up((((size_t)k << (k - 1)) * (size_t)L + (ct_comp_in_lds(L, k) ? 0 : CtLds::comp_count(L, k))) * 4, 256);
}

hipError_t launch_ct_solve(const float* t, const float* m, const float* w, const float* M, const float* v, const float* B, int L,
                           int k, int n_inst, float* beta_out, int32_t* cuts_out, int32_t* order_out, void* slots,
                           size_t slot_count, hipStream_t stream) {
    const bool in_lds = ct_comp_in_lds(L, k);
    const int H = L <= 64 ? 1 : 2;
    const uint32_t lds_bytes = CtLds::make(L, k, H, kCtWaves, in_lds).total;
    const uint32_t grid = (uint32_t)(slot_count < (size_t)n_inst ? slot_count : (size_t)n_inst);
    auto launch = [&](auto kernel, std::atomic<uint64_t>& lds_allowed) -> hipError_t {
        const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(kernel), lds_allowed);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kCtWaves * 64), lds_bytes, stream, t, m, w, M, v, B, L, k, n_inst, beta_out,
                           cuts_out, order_out, static_cast<uint32_t*>(slots), ct_slot_bytes(L, k) / 4);
        return hipGetLastError();
    };
    static std::atomic<uint64_t> allowed[4];
    if (in_lds) return H == 1 ? launch(&ct_solve_kernel<1, true>, allowed[0]) : launch(&ct_solve_kernel<2, true>, allowed[1]);
    return H == 1 ? launch(&ct_solve_kernel<1, false>, allowed[2]) : launch(&ct_solve_kernel<2, false>, allowed[3]);
}

hipError_t launch_ct_tables(const float* t, const float* m, const float* w, const float* M, const float* v, const float* B,
                            int L, int k, int n_inst, void* ws, hipStream_t stream) {
    const CtLayout y = CtLayout::make(L, k);
    hipLaunchKernelGGL(ct_tables_kernel, dim3(n_inst), dim3(kCtPreThreads), 0, stream, t, m, w, M, v, B, y,
                       static_cast<unsigned char*>(ws));
    return hipGetLastError();
}

// beta of every ordering of one instance with rank in [rank_begin, rank_end)
hipError_t launch_ct_enumerate(int L, int k, const void* ws, uint32_t rank_begin, uint32_t rank_end, float* beta_export,
                               hipStream_t stream) {
    const uint32_t span = rank_end - rank_begin;
    if (span == 0) return hipSuccess;
    const CtLayout y = CtLayout::make(L, k);
    // a lane's row takes (L + 1) words of LDS: 256 lanes per workgroup where that fits beside the tables, else 128
    int threads = 256;
    if ((size_t)y.ct_off + (size_t)(L + 1) * threads * 4 > (size_t)kLdsBytesPerCU) threads = 128;
    const size_t lds = (size_t)y.ct_off + (size_t)(L + 1) * threads * 4;
    if (lds > (size_t)kLdsBytesPerCU) return hipErrorInvalidValue;
    uint32_t gx = (span + threads - 1) / threads;
    if (gx > 4096u) gx = 4096u;
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&ct_enumerate_kernel), lds_allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ct_enumerate_kernel, dim3(gx), dim3(threads), lds, stream, y, static_cast<const unsigned char*>(ws),
                       rank_begin, rank_end, beta_export);
    return hipGetLastError();
}

}  // namespace ppo
