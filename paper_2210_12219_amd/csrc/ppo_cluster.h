// Layout of the cluster form's tables, shared by the kernels that make them and those that search.
#pragma once

#include "ppo_common.h"

namespace ppo {

// Codes as in the fixed-k kernels: kCodeZero for the value 0 (also that of a link: with the number of segments free it ties
// with a segment that needs none), kCodeZero + 1 + #{smaller quotients}, kCodeInf for +inf: positive normal binary16 patterns, so the three-input binary16 minimum acts as an integer minimum.
// Everything these kernels read as a code is written by them as one (a stray pattern could win that minimum).
constexpr uint32_t kClZero = kCodeZero, kClInf = kCodeInf;
constexpr int kClPreThreads = 1024;
static_assert((int)kClZero + (PPO_CLUSTER_MAX_N * (PPO_CLUSTER_MAX_N - 1) / 2) * (PPO_MAX_L - 1) + 1 < (int)kClInf,
              "codes stay below +inf");
static_assert(((unsigned long long)PPO_CLUSTER_MAX_N << (PPO_CLUSTER_MAX_N - 1)) * ((PPO_MAX_L + 1) / 2) < (1ull << 32),
              "the dwords of one instance's rows are counted in 32 bits");

// How the level kernel lays rows over lanes: chains of up to 63 layers (their rows with the entry of the chain's end fit 32
// lanes of two entries) go two sets to a wave; up to 127 one set; 128 layers one set, with an entry beyond the lanes.
enum { kClTwoSets = 0, kClOneSet = 1, kClWide = 2 };
__host__ __device__ constexpr int cluster_mode(int L) { return L <= 63 ? kClTwoSets : L <= 127 ? kClOneSet : kClWide; }
__host__ __device__ constexpr int cluster_sets_per_wave(int mode) { return mode == kClTwoSets ? 2 : 1; }
// Run minima of a wave: rows of kClRunPitch dwords for runs of 2^0, 2^1 .. entries, then entries that are +inf, for windows
// that are empty (two sets: the second one's lie 32 dwords on).
__host__ __device__ constexpr int cluster_run_pitch(int mode) { return mode == kClWide ? 80 : 64; }
__host__ __device__ constexpr int cluster_run_levels(int mode) { return mode == kClTwoSets ? 6 : 7; }
__host__ __device__ constexpr int cluster_run_dwords(int mode) {
    return cluster_run_levels(mode) * cluster_run_pitch(mode) + (mode == kClTwoSets ? 36 : 4);
}
// A search on fewer nodes and cuts: four to eight sets to a wave on up to 31 layers, which have runs of up to 16 entries and
// the +inf in the row of the next longer ones, up to 56 dwords on; else two sets.
__host__ __device__ constexpr int cluster_part_none(int L) { return (L <= 31 ? 5 : 6) * 64; }

struct ClusterLayout {
    int L, n, npairs, nq, rs;                       // rs: entries per row of A: 0..L-1 (entry L is never finite
                                                    // and not stored), rounded up to even
    uint32_t hi_off, qc_off, dec_off, qv_off, ord_off, img_off, stride;   // bytes within one instance's tables
    bool may_be_reduced;                            // the call's instances may be searched on fewer nodes and cuts

    __host__ __device__ static ClusterLayout make(int L, int n, bool may_be_reduced = false) {
        ClusterLayout y;
        y.may_be_reduced = may_be_reduced;
        y.L = L;
        y.n = n;
        y.npairs = n * (n - 1) / 2;
        y.nq = y.npairs * (L - 1);
        y.rs = (L + 1) & ~1;
        size_t off = 0;
        y.hi_off = (uint32_t)off;
        off = align_up(off + (size_t)n * (L + 1), 16);
        y.qc_off = (uint32_t)off;
        off = align_up(off + (size_t)y.npairs * L * 2, 16);
        y.dec_off = (uint32_t)off;
        off = align_up(off + ((size_t)y.nq + 1) * 4, 16);
        y.qv_off = (uint32_t)off;
        off = align_up(off + (size_t)y.nq * 4, 16);
        y.ord_off = (uint32_t)off;   // the layers 0 .. L-2 in increasing order of t (one byte each)
        off = align_up(off + (size_t)L, 256);
        // what the level kernel keeps in LDS, ready to be copied: quotient rows (rs / 2 dwords each, the pitch of the rows
        // of A), then the window queries of every (node, entry); and the longest run that a query asks for
        y.img_off = (uint32_t)off;
        off = align_up(off + y.q_image_bytes() + y.query_bytes() + 16, 256);
        y.stride = (uint32_t)off;
        return y;
    }
    // bytes of the quotient rows in the LDS image (the window queries follow, 16-byte aligned): two sets to a wave, of
    // every ordered pair, so that a lane finds the row of (j, j'') by one addition; one set, of every pair a < b, at
    // below(b) + a (half the space, and the offset is the wave's)
    __host__ __device__ size_t q_image_bytes() const {
        return align_up((size_t)(cluster_mode(L) == kClTwoSets ? n * n : npairs) * (rs / 2) * 4, 16);
    }
    __host__ __device__ size_t query_bytes() const { return (size_t)n * (128 / cluster_sets_per_wave(cluster_mode(L))) * 4; }
    // Where an instance that is searched on fewer nodes and cuts says so (ppo_cluster_bound.hip): a flag behind the longest
    // run, and in what is then free of the image, as the tables are those of a smaller layout, which nodes and cuts.
    __host__ __device__ size_t flag_off() const { return img_off + q_image_bytes() + query_bytes() + 4; }
    __host__ __device__ size_t record_off() const { return (img_off + q_image_bytes() + query_bytes() - 32) & ~(size_t)7; }
    // pair a < b is row below(b) + a.  below(j) + m > below(m) + j for m < j, so that the larger of the two is the row of
    // the pair in either order (the value for node 0, which is never the larger one, is chosen for that).
    __host__ __device__ static constexpr int below(int b) { return b ? (int)((uint32_t)(b * (b - 1)) >> 1) : -2; }
    // rows A[R][j] exist for j in R only: n 2^(n-1) of them per instance
    __host__ __device__ size_t rows_per_instance() const { return (size_t)n << (n - 1); }
    __host__ __device__ size_t rows_bytes() const { return rows_per_instance() * (size_t)rs * sizeof(uint16_t); }
};

constexpr size_t kClBinomialBytes = (size_t)(PPO_CLUSTER_MAX_N + 1) * (PPO_CLUSTER_MAX_N + 1) * 4;   // in LDS, of the levels of such an instance

// Nodes and cuts (bit e: the cut e) that an instance's tables are made of, if not of all.
struct ClusterRecord {
    unsigned long long cuts[2];
    uint32_t nodes;
};
static_assert(sizeof(ClusterRecord) <= 32, "the record lies in the last 32 bytes of the image");

// What the tables at `base` (of an instance whose slice has the layout `whole`) are made of.  The flag is always written.  The
// kernels that run once a call do not read it where the call says that everything is searched (calls with one segment, which have
// one level); the levels just read it: asking first made every level of a confined search 0.1 to 0.2 us longer (one cluster of 20
// nodes 316 us a call so, 320 without the question anywhere, 1.3 % more with it in the levels too; 32 of 15 nodes 494, 493 and 497).
__device__ __forceinline__ bool cluster_flag(const ClusterLayout& whole, const unsigned char* base) {
    return __builtin_amdgcn_readfirstlane(*reinterpret_cast<const int*>(base + whole.flag_off())) != 0;
}
__device__ __forceinline__ bool cluster_reduced(const ClusterLayout& whole, const unsigned char* base) {
    return whole.may_be_reduced && cluster_flag(whole, base);
}
__device__ __forceinline__ ClusterLayout cluster_part_layout(const ClusterLayout& whole, const unsigned char* base) {
    const ClusterRecord r = *reinterpret_cast<const ClusterRecord*>(base + whole.record_off());
    return ClusterLayout::make(__builtin_amdgcn_readfirstlane(__popcll(r.cuts[0]) + __popcll(r.cuts[1]) + 1),
                               __builtin_amdgcn_readfirstlane(__popc(r.nodes)));
}
__device__ __forceinline__ ClusterLayout cluster_layout(const ClusterLayout& whole, const unsigned char* base) {
    return cluster_reduced(whole, base) ? cluster_part_layout(whole, base) : whole;
}

// Tables of an instance on the nodes and cuts that can matter, where every node may be used or not: what
// cluster_tables_kernel does otherwise.
hipError_t launch_cluster_reduce(const float* t, const float* m, const float* M, const float* B, const ClusterLayout& y, int n_inst,
                                 unsigned char* ws, hipStream_t stream);

// The same for the search for few segments: two bounds, then whether the search is confined, and to which nodes and cuts.
struct FewConfined {
    union {
        uint32_t bounds[2];
        unsigned long long nodes;
    };
    unsigned long long cuts[2];
    uint32_t in, bound;   // no value above the bound matters (+inf: none is known)
};
// `out`: of the first instance, `stride` bytes to that of the next
hipError_t launch_few_confine(const float* t, const float* m, const float* M, const float* B, int L, int n, int pmax, int n_inst,
                              FewConfined* out, size_t stride, hipStream_t stream);

}  // namespace ppo
