// Dynamic programming over the sets of nodes not yet used, on the cuts that a set can meet: the second stage of the staged
// search by subsets (ppo_solve_subsets), and ppo_solve for many instances of long chains.
//
// The bottleneck of Eq. 2 is a maximum over links, so what is still to be paid from a cut on depends only on the
// node j that takes the next segment, the cut e and the set R of nodes not used before it (j in R):
//     A[{j}][j][e] = 0 if layers [e, L) fit node j, else +inf
//     A[R][j][e]   = min over e' in (e, min(hi_j(e), L-1)] of  min over j'' in R' of max(q_{j,j''}[e'-1], A[R'][j''][e'])
// with R' = R \ j and hi_j(e) the last e' such that layers [e, e') fit node j; beta* = min over j of A[All][j][0].
// k 2^(k-1) rows replace the k! programmes of the enumeration.  The rows are those of the cluster form
// (ppo_cluster.hip) with every node to be used.
//
// Ranges.  Every node is used and memory is tight, so the cut before the last |R| segments cannot lie just anywhere: the
// nodes of R have to hold the layers after it and the others those before it.  With
//     most[S]  = an upper bound of the layers from the start that S holds in any order
//     least[S] = a lower bound of the cuts from which S holds the rest
// the rows of R matter only for e in [max(least[R], k - |R|), min(most[All \ R], L - |R|)].  Below that range every entry is
// +inf; above it no prefix arrives, so windows may stop at its end.  Capacities of 1.25 of the model leave 20 to 25 entries of
// 96, of 1.3 10 to 45 of 50 to 127.  A row is held from an even entry at or before its range, and a wave takes eight, four,
// two or one sets, as many as the widest ranges of the level allow (16, 32, 64 or 128 entries).  With ample memory a range is
// nearly the chain, and there is nothing to gain: see bands_whole_rows.
//
// Values.  The rows hold 16-bit codes that do not decrease with the quotient: kCodeZero for 0, then kCodeZero + 1 +
// ((bits - lo) >> shift) with [lo, hi] the range of the quotients' binary32 patterns and the least shift that fits, and
// kCodeInf beyond.  Minima and maxima commute with a non-decreasing map, so the search gives the code of beta*.  If
// more than one of the quotients has that code, the search is repeated with [lo, hi] the range of those (everything
// below counts as 0, everything above as +inf): a pass divides the range by 30,000, so there are at most three, and
// after the last one "code <= code of beta*" says the same as "value <= beta*".
//
// What bounds it: instruction issue.  4096 x (96, 8) take 35,000 vector and 21,000 scalar instructions an instance, about half
// of them in the levels (75 vector instructions for four rows of 25 entries, where a row of 96 took 47 by itself); the rest is
// what every wave of a workgroup works out for itself in each phase, and it grows with the waves.  The phases that one wave
// or a few work alone (sums, windows, answer) overlap with those of the other workgroups of the compute unit.
// Measured, before and now: 4096 x (96, 8) of transformers 624 / 347 to 354 us, of random chains 739 / 583, 1024 x (65, 8) 218 / 143,
// 4096 x (80, 6) 311 / 227; staged (tables and final stage included) 64 x (100, 10) 260 / 197, 1024 x (50, 6) 180 / 125, 300 x
// (20, 10) 313 / 159.  (Memory of 1.2 to 1.3 times what the chain needs; of twice and four times: bands_whole_rows.)
#include "ppo_sets.h"

namespace ppo {

static __constant__ SetValues kSetValues = SetValues();

namespace {

constexpr uint32_t kFinestCodes = kCodeInf - kCodeZero - 2u;   // buckets of the code
constexpr int kSubsetMaxWaves = 16;
constexpr int kSmallK = 8;   // up to as many nodes one workgroup does the whole search of an instance

// G sets share a wave, 64 / G lanes of two entries each.  Minima over runs of 2^r entries of a wave's rows: a row of 64
// dwords per r, up to half the entries of a set.  One set: runs of 64 are asked for at the first 65 of its entries only, so the
// last row is shorter, with a dword for what the other lanes write; then entries that are +inf, for windows that are empty.
__host__ __device__ constexpr int run_levels(int G) { return G == 1 ? 7 : G == 2 ? 6 : G == 4 ? 5 : 4; }
constexpr uint32_t kLastRun = 33u, kRunNone = 6u * 64u + kLastRun + 1u;   // the dword, and the first of those entries
__host__ __device__ constexpr uint32_t run_dwords(int G) { return G == 1 ? kRunNone + 8u : (uint32_t)run_levels(G) * 64u; }
// A search on whole rows (bands_whole_rows) answers windows from a table of queries.
__host__ __device__ constexpr uint32_t query_pitch(int L) { return (uint32_t)(L + 2) & ~1u; }   // dwords of a node
__host__ __device__ constexpr uint32_t query_bytes(int L, int k) { return L - k + 2 > 64 ? (uint32_t)k * query_pitch(L) * 4u : 0u; }

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef short ss2 __attribute__((ext_vector_type(2)));
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

// Reductions over a wave by lane shifts (rows of 16, then the last lane of a row to the next row, of two rows to the next
// two): the result of lane 63, in all lanes.
#define PPO_WAVE_STEPS(op, none)                                                                                          \
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)v, 0x111, 0xF, 0xF, false));                        \
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)v, 0x112, 0xF, 0xF, false));                        \
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)v, 0x114, 0xF, 0xF, false));                        \
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)v, 0x118, 0xF, 0xF, false));                        \
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)v, 0x142, 0xA, 0xF, false));                        \
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)v, 0x143, 0xC, 0xF, false));                        \
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
__device__ __forceinline__ uint32_t larger(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t smaller(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t either(uint32_t a, uint32_t b) { return a | b; }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) { PPO_WAVE_STEPS(larger, 0u) }
__device__ __forceinline__ uint32_t wave_min(uint32_t v) { PPO_WAVE_STEPS(smaller, ~0u) }
__device__ __forceinline__ uint32_t wave_or(uint32_t v) { PPO_WAVE_STEPS(either, 0u) }
#undef PPO_WAVE_STEPS

struct BandsShared {
    uint32_t lo_bits, hi_bits;                 // range of the quotients that get codes of their own
    uint32_t bucket_lo, bucket_hi;
    uint32_t over16, over32, over64;           // bit c: a set of c nodes has a range of more than 16 (32, 64) entries
    uint32_t widest;                           // entries of the widest range
    uint32_t whole, longest;                   // whole rows; log2 of the longest run that a window is then made of
    uint32_t level[PPO_MAX_K + 2];             // first entry of the sets of every size in `order`
};

// A set's entry of `info`: its first row, the (even) entry its rows start at, the last of its range, and whether that is
// empty.
constexpr uint32_t kEmptySet = 1u << 31;
__device__ __forceinline__ uint32_t info_row(uint32_t info) { return info & 0x7FFFu; }
__device__ __forceinline__ int info_base(uint32_t info) { return (int)((info >> 14) & 0x7Eu); }
__device__ __forceinline__ int info_end(uint32_t info) { return (int)((info >> 21) & 0x7Fu); }
__device__ __forceinline__ uint32_t make_info(uint32_t row, int base, int end) { return row | (uint32_t)base << 14 | (uint32_t)end << 21; }
static_assert((PPO_MAX_K << (PPO_MAX_K - 1)) <= 0x8000 && PPO_MAX_L <= 128, "rows and cuts fit their fields");
__device__ __forceinline__ uint32_t mul24(uint32_t a, uint32_t b) { return __umul24(a, b); }

// LDS (byte offsets), all of it in the dynamic part (the limit of that part is raised to all there is).  What lies before
// run_off is kept between the launches of a search that takes several, as an image behind the rows.
struct BandsLds {
    uint32_t info_off, order_off, P_off, t_off, B_off, M_off, hi_off, lo_off, q_off, run_off;
    int hp, qp;                                // pitch of a row of hi and lo (bytes), of quotient codes (dwords)
    __host__ __device__ static BandsLds make(int L, int k, bool raw) {
        BandsLds s;
        size_t off = align_up(sizeof(BandsShared), 16);
        s.info_off = (uint32_t)off;                      // [2^k] u32
        off += (size_t)4 << k;
        s.order_off = (uint32_t)off;                     // [2^k] u16: the sets in increasing order of size, then of value
        off = align_up(off + ((size_t)2 << k), 16);
        s.P_off = (uint32_t)off;                         // written 64 at a time
        off = align_up(off + (align_up((size_t)L, 64) + 1) * 8, 16);
        s.t_off = (uint32_t)off;
        off = align_up(off + (size_t)L * 4, 16);
        s.B_off = (uint32_t)off;
        off = align_up(off + (size_t)k * k * 4, 16);
        s.M_off = (uint32_t)off;
        off = align_up(off + (size_t)k * 4, 16);
        s.hp = (L + 3) & ~1;
        s.hi_off = (uint32_t)off;
        off = align_up(off + (size_t)k * s.hp, 16);
        s.lo_off = (uint32_t)off;
        off = align_up(off + (raw ? 0 : (size_t)k * s.hp) + 128, 16);   // lanes beyond a row of hi read on, and drop what they read
        s.qp = (L + 1) / 2;
        s.q_off = (uint32_t)off;                         // [k][k] rows: entry e of (j, j'') belongs to the cut e
        off = align_up(off + ((size_t)k * k * s.qp + 64) * 4, 256);
        s.run_off = (uint32_t)off;
        return s;
    }
};

// dwords of the rows of an instance in global memory, a multiple of 256 bytes
__host__ __device__ inline uint32_t row_dwords(int k, int rd) { return (((uint32_t)k << (k - 1)) * (uint32_t)rd + 63u) & ~63u; }
// ... of an area: no range is longer.  Sets of c < k nodes are met at cuts from k - c to L - c, the set of all at up to L - k, and
// a row starts at an even cut.
__host__ __device__ inline uint32_t area_dwords(int k, int L) { return row_dwords(k, (L - k + 3 < L + 1 ? L - k + 3 : L + 1) / 2); }

// What the levels of an instance work on.
struct BandsCtx {
    const uint32_t* q32;
    const unsigned char* hi_s;
    const uint32_t* info;
    const uint16_t* order;                     // the sets of the level's size
    int L, k, rd, hp, qp;                      // rd: dwords of a row
};

// Rows A[R' + j][j] of every set R' of C nodes (C >= 1) and every j outside it.  An item of work is a group of G sets and
// one part in 2^split of the nodes outside (so that levels of few sets keep all waves busy); wave `wave` of `waves`.
template <int C, int G>
__device__ __forceinline__ void bands_level(const BandsCtx c, int lane, int wave, int waves, int split, uint32_t nsets,
                                             uint32_t* __restrict__ run32, uint32_t* rows) {
    constexpr int kLanes = 64 / G;
    constexpr uint32_t kInf2 = kCodeInf | (kCodeInf << 16);
    const int hl = lane & (kLanes - 1), part = lane / kLanes, rd = c.rd, k = c.k;
    const int hload = hl < rd ? hl : rd - 1;   // lanes beyond a row read its last dword
    const uint32_t all = (1u << k) - 1u, q_node = (uint32_t)c.qp * 4u;   // bytes from the link of one node to that of the next
    const int outside = k - C, per = (outside + (1 << split) - 1) >> split;
    const int items = (int)((nsets + (uint32_t)G - 1u) / (uint32_t)G) << split;
    // a lane's place in a row of hi, of the links and of its run minima
    const uint32_t hi_at = 2u * (uint32_t)hl;
    const int last_at = lane < (int)kLastRun ? lane : (int)kLastRun;   // in the row of the longest runs
    unsigned char* runb = reinterpret_cast<unsigned char*>(run32) + part * (kLanes * 4);
    auto put_row = [&](uint32_t up, uint32_t set, uint32_t j, uint32_t value) {   // a byte offset of 32 bits
        const uint32_t row = info_row(up) + (uint32_t)__popc(set & ((1u << j) - 1u));
        *reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(rows) + ((mul24(row, (uint32_t)rd) + (uint32_t)hl) << 2)) = value;
    };
    for (int it = wave; it < items; it += waves) {
        const int skip = (it & ((1 << split) - 1)) * per;
        const int count = outside - skip < per ? outside - skip : per;
        if (count <= 0) continue;
        uint32_t idx = (uint32_t)(it >> split) * (uint32_t)G + (uint32_t)part;
        const bool mine = idx < nsets;
        if (G > 1 && !mine) idx = nsets - 1u;
        uint32_t mp = c.order[idx], info = c.info[mp];
        if (G == 1) {
            mp = (uint32_t)__builtin_amdgcn_readfirstlane((int)mp);
            info = (uint32_t)__builtin_amdgcn_readfirstlane((int)info);
        }
        uint32_t jb = all & ~mp;
        for (int i = 0; i < skip; ++i) jb &= jb - 1u;
        const bool empty = (info & kEmptySet) != 0u, writes = hl < rd && mine;
        if (__ballot(!empty) == 0ull) {
            // nothing can be done from these sets: rows of the sets above whose ranges are not empty are +inf
            for (int i = 0; i < count; ++i, jb &= jb - 1u) {
                const uint32_t j = (uint32_t)__ffs(jb) - 1u, set = mp | (1u << j), up = c.info[set];
                if (writes && !(up & kEmptySet)) put_row(up, set, j, kInf2);
            }
            continue;
        }
        const int base = info_base(info);
        uint32_t a[C], qoff[C];
        {
            const uint32_t* arow = rows + mul24(info_row(info), (uint32_t)rd) + (uint32_t)hload;
            uint32_t bits = mp;
#pragma unroll
            for (int m = 0; m < C; ++m) {
                qoff[m] = mul24((uint32_t)(__ffs(bits) - 1), (uint32_t)k * q_node) + (uint32_t)((base >> 1) + hl) * 4u;
                bits &= bits - 1u;
                a[m] = empty ? kInf2 : arow[m * rd];
            }
        }
        // Local entry that windows may end at.  Entries beyond a set's range need not have been written.
        const short last = (short)(info_end(info) - base);
        uint32_t up = c.info[mp | (jb & (0u - jb))];
        for (int i = 0; i < count; ++i) {
            const uint32_t bit = jb & (0u - jb), set = mp | bit;
            const uint32_t j = (uint32_t)__ffs(jb) - 1u;
            jb ^= bit;
            const int ubase = info_base(up);
            const uint32_t h01 = *reinterpret_cast<const uint16_t*>(c.hi_s + mul24(j, (uint32_t)c.hp) + (uint32_t)ubase + hi_at);
            uint32_t v;
            {
                const uint32_t qj = mul24(j, q_node);
                uint32_t x[C];
#pragma unroll
                for (int m = 0; m < C; ++m)
                    x[m] = pk_max(*reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(c.q32) + qoff[m] + qj), a[m]);
                v = x[0];
#pragma unroll
                for (int m = 1; m + 1 < C; m += 2) v = pk_min3(v, x[m], x[m + 1]);
                if (C % 2 == 0) v = pk_min(v, x[C - 1]);
            }
            const uint32_t up_now = up;
            up = c.info[mp | (jb & (0u - jb))];   // of the next node (or of R' itself, and dropped)
            // minima over runs of 2^r entries starting at each entry; a run that passes the end of the row holds
            // whatever lies there and is never asked for (shifts towards lower lanes; four and eight sets: within 16 lanes)
            constexpr int kUp1 = G >= 4 ? 0x101 : 0x130;
            run32[lane] = v;
            const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kUp1, 0xF, 0xF, true);
            uint32_t cur = pk_min(v, (v >> 16) | (next << 16));
            run32[64 + lane] = cur;
            cur = pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, kUp1, 0xF, 0xF, true));
            run32[128 + lane] = cur;
            if (G >= 4) {
                cur = pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x102, 0xF, 0xF, true));
                run32[192 + lane] = cur;
                if (G == 4) {
                    cur = pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x104, 0xF, 0xF, true));
                    run32[256 + lane] = cur;
                }
            } else {
                const uint32_t s1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x130, 0xF, 0xF, true);
                cur = pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)s1, 0x130, 0xF, 0xF, true));
                run32[192 + lane] = cur;
#pragma unroll
                for (int r = 4; r < run_levels(G); ++r) {
                    if (2 * rd <= (1 << r)) break;   // no window takes a run as long as a row
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    cur = pk_min(cur, run32[(r - 1) * 64 + ((lane + (1 << (r - 2))) & 63)]);
                    run32[r * 64 + (r == 6 ? last_at : lane)] = cur;
                }
            }
            // The window of entry e (of R' + j's rows) in entries of R's: from max(e + 1, base) to min(hi, last); two
            // runs of 2^r entries cover it, 2^r the largest power of two below its length (or 1).  Empty: `none` is +inf.
            const short from = (short)(ubase - base + 2 * hl + 1);
            const ss2 start = __builtin_elementwise_max(ss2{from, (short)(from + 1)}, ss2{0, 0});
            const ss2 end = __builtin_elementwise_min(ss2{(short)((int)(h01 & 0xFFu) - base), (short)((int)(h01 >> 8) - base)}, ss2{last, last});
            const ss2 over = end - start;
            const uint32_t none = __builtin_bit_cast(uint32_t, over >> 15) & kInf2;
            const ss2 more = __builtin_elementwise_max(over, ss2{0, 0});
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint32_t r1[2], r2[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t d = (uint16_t)(h ? more.y : more.x), s = (uint16_t)(h ? start.y : start.x);
                const uint32_t r = 31u - (uint32_t)__builtin_clz(d | 1u);
                const uint32_t at = (r << 8) + 2u * s;
                r1[h] = *reinterpret_cast<const uint16_t*>(runb + at);
                r2[h] = *reinterpret_cast<const uint16_t*>(runb + at + 2u * (d + 1u - (1u << r)));
            }
            const uint32_t res = pk_max(pk_min(r1[0] | (r1[1] << 16), r2[0] | (r2[1] << 16)), none);
            if (writes && !(up_now & kEmptySet)) put_row(up_now, set, j, res);
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// First cut of a row of a set of c nodes, with whole rows.
__device__ __forceinline__ int whole_base(int k, int c) { return (k - c) & ~1; }

// The same with whole rows, one set to a wave: all rows of a level start at the same cut, so windows are looked up in a table
// (`query`, see bands_queries).
template <int C>
__device__ __forceinline__ void bands_level_whole(const BandsCtx c, int lane, int wave, int waves, int split, uint32_t nsets,
                                                   const uint32_t* query, int run_top, uint32_t* __restrict__ run32, uint32_t* rows) {
    constexpr uint32_t kInf2 = kCodeInf | (kCodeInf << 16);
    const int rd = c.rd, k = c.k;
    const bool in_row = lane < rd;
    const int hq = in_row ? lane : rd - 1;     // lanes beyond a row look up its last window, and drop the answer
    const int base = whole_base(k, C), ubase = whole_base(k, C + 1);
    const uint32_t all = (1u << k) - 1u;
    const int outside = k - C, per = (outside + (1 << split) - 1) >> split;
    const int items = (int)nsets << split;
    const int last_at = lane < (int)kLastRun ? lane : (int)kLastRun;
    if (lane < 8) run32[kRunNone + (uint32_t)lane] = kInf2;
    // the table holds places among entries that start at the cut 0
    const unsigned char* runb = reinterpret_cast<const unsigned char*>(run32) - 2 * base;
    const uint32_t* my_query = query + ubase + 2 * hq;
    const uint32_t query_node = query_pitch(c.L), q_node = (uint32_t)c.qp * 4u;
    // A row that starts two cuts before those it is made of has a first entry that no placement reaches (too few layers
    // come before it); what it looks up is not one of the entries.
    const uint32_t unreached = lane == 0 && base != ubase ? kCodeInf : 0u;
    for (int it = wave; it < items; it += waves) {
        const int skip = (it & ((1 << split) - 1)) * per;
        const int count = outside - skip < per ? outside - skip : per;
        if (count <= 0) continue;
        const uint32_t mp = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.order[it >> split]);
        const uint32_t first_row = info_row((uint32_t)__builtin_amdgcn_readfirstlane((int)c.info[mp]));
        uint32_t jb = all & ~mp;
        for (int i = 0; i < skip; ++i) jb &= jb - 1u;
        uint32_t a[C], qoff[C];
        {
            const uint32_t* arow = rows + first_row * (uint32_t)rd + (uint32_t)hq;
            uint32_t bits = mp;
#pragma unroll
            for (int m = 0; m < C; ++m) {
                qoff[m] = (uint32_t)(__ffs(bits) - 1) * (uint32_t)k * q_node + (uint32_t)((base >> 1) + lane) * 4u;
                asm volatile("" : "+v"(qoff[m]));   // one addition per row and member: the scalar unit has enough to do
                bits &= bits - 1u;
                const uint32_t x = arow[m * rd];
                a[m] = in_row ? x : kInf2;
            }
        }
        // where the rows of this set go: lane j works it out for the node j (the scalar unit has enough to do)
        const uint32_t out_off = mul24(row_of(first_row, mp, (uint32_t)lane & 15u), (uint32_t)rd);
        for (int i = 0; i < count; ++i, jb &= jb - 1u) {
            const uint32_t j = (uint32_t)__ffs(jb) - 1u;
            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)out_off, (int)j);
            const uint2 qd = *reinterpret_cast<const uint2*>(my_query + j * query_node);
            uint32_t v;
            {
                uint32_t x[C];
                const unsigned char* qj = reinterpret_cast<const unsigned char*>(c.q32) + j * q_node;
#pragma unroll
                for (int m = 0; m < C; ++m) x[m] = pk_max(*reinterpret_cast<const uint32_t*>(qj + qoff[m]), a[m]);
                v = x[0];
#pragma unroll
                for (int m = 1; m + 1 < C; m += 2) v = pk_min3(v, x[m], x[m + 1]);
                if (C % 2 == 0) v = pk_min(v, x[C - 1]);
            }
            run32[lane] = v;
            const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xF, 0xF, true);
            uint32_t cur = pk_min(v, (v >> 16) | (next << 16));
            run32[64 + lane] = cur;
            cur = pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x130, 0xF, 0xF, true));
            run32[128 + lane] = cur;
            const uint32_t s1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)cur, 0x130, 0xF, 0xF, true);
            cur = pk_min(cur, (uint32_t)__builtin_amdgcn_mov_dpp((int)s1, 0x130, 0xF, 0xF, true));
            run32[192 + lane] = cur;
#pragma unroll
            for (int r = 4; r < run_levels(1); ++r) {
                if (r > run_top) break;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                cur = pk_min(cur, run32[(r - 1) * 64 + ((lane + (1 << (r - 2))) & 63)]);
                run32[r * 64 + (r == 6 ? last_at : lane)] = cur;
            }
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
            if (in_row)   // a byte offset of 32 bits
                *reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(rows) + ((row + (uint32_t)lane) << 2)) =
                    (unreached ? kCodeInf : res[0]) | (res[1] << 16);
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Where an instance comes from and where its answer goes: arrays of the problem, and beta, cuts and order; or the tables
// of ppo_prepare (window starts, exact codes, the codes' values), and the key.
struct BandsTask {
    const float *t, *m, *M, *B;
    const unsigned char* prepared;
    Layout y;
    float* beta;
    int32_t *cuts, *order;
    unsigned long long* key;
    uint32_t* slots;            // row areas in global memory
    uint32_t slot_dwords;
    uint32_t lds_bytes;         // of the launch
    uint32_t query_bytes;       // of the levels that are launches: for the table of whole rows; 0: there is no room for it
    int L, k, n_inst, from, to;
    // log2 of the parts of the nodes outside, by level: 4 bits, two sets to a wave (or one), then four; 2 bits, whole rows
    unsigned long long splits;
    uint32_t whole_splits;
};

// A level with as many sets to a wave as its ranges allow.
template <int C>
__device__ __forceinline__ void bands_level_any(const BandsShared& sh, BandsCtx c, const uint16_t* order, int lane, int wave,
                                                 int waves, const BandsTask& task, const uint32_t* query, uint32_t* run32,
                                                 uint32_t* rows) {
    // nothing of a level is worked out before it: values of all levels and forms, hoisted, do not fit the registers
    asm volatile("" : "+v"(lane), "+s"(wave), "+s"(c.k), "+s"(c.rd), "+s"(c.qp));
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.level[C]);
    const uint32_t nsets = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.level[C + 1]) - first;
    const uint32_t here = 3u << C;   // the rows read and the rows written
    c.order = order + first;
    const int s = (int)(task.splits >> (4 * C));
    if (sh.whole)
        bands_level_whole<C>(c, lane, wave, waves, (int)(task.whole_splits >> (2 * C)) & 3, nsets, query, (int)sh.longest, run32, rows);
    else if (sh.over64 & here)
        bands_level<C, 1>(c, lane, wave, waves, s & 3, nsets, run32, rows);
    else if (sh.over32 & here)
        bands_level<C, 2>(c, lane, wave, waves, s & 3, nsets, run32, rows);
    else if (sh.over16 & here)
        bands_level<C, 4>(c, lane, wave, waves, (s >> 2) & 3, nsets, run32, rows);
    else
        bands_level<C, 8>(c, lane, wave, waves, (s >> 2) & 3, nsets, run32, rows);
}

// nodes a < b of pair p in row-major order of the pairs
__device__ __forceinline__ void pair_nodes(int p, int k, int& a, int& b) {
    a = 0;
    while (p >= k - 1 - a) { p -= k - 1 - a; ++a; }
    b = a + 1 + p;
}

// entry `cut` of the rows of (a, b) and (b, a)
__device__ __forceinline__ void put_code(uint16_t* q16, int k, int qp, int a, int b, int cut, uint32_t code) {
    q16[(a * k + b) * (2 * qp) + cut] = (uint16_t)code;
    q16[(b * k + a) * (2 * qp) + cut] = (uint16_t)code;
}

}  // namespace

// Part of the search that a launch does: all of it, or (many nodes and few instances: the widest levels are launches of
// their own, see launch_bands_keys) the tables and the levels up to `from`, or those from `to` on and what follows them.
enum { kWhole = 0, kHead = 1, kTail = 2 };

// What the phases of the kernel share: an instance's tables in LDS.  Every phase works its own view out, from values that
// are opaque to the compiler, so that nothing is held in registers from one phase to the next: hoisted out of the loop
// over instances, the addresses and comparisons of all phases do not fit them, and what is then reloaded from scratch memory
// made the phases of one wave twice as long.
struct BandsView {
    int tid, lane, wave, waves, threads, L, k, hp, qp, npairs, rd;
    uint32_t all;
    BandsShared& sh;
    uint32_t* info;
    uint16_t* set_order;
    double* P;
    float *t_s, *B_s, *M_s;
    unsigned char *hi_s, *lo_s;
    uint16_t* q16;
    unsigned char* scratch;     // before the levels
    uint32_t *run32, *query, *lds_rows, *slot;
    bool raw, in_lds;
    const unsigned char* prep;

    __device__ __forceinline__ static int opaque(int x) {
        asm volatile("" : "+s"(x));
        return x;
    }
    __device__ __forceinline__ static int opaque_lane(int x) {
        asm volatile("" : "+v"(x));
        return x;
    }
    __device__ __forceinline__ BandsView(unsigned char* sm, const BandsTask& task, uint32_t inst, bool is_raw, bool may_use_lds)
        : tid(opaque_lane((int)threadIdx.x)), lane(tid & 63), wave(__builtin_amdgcn_readfirstlane(tid >> 6)),
          waves(opaque((int)blockDim.x >> 6)), threads(waves * 64), L(opaque(task.L)), k(opaque(task.k)),
          sh(*reinterpret_cast<BandsShared*>(sm)) {
        const BandsLds lds = BandsLds::make(L, k, is_raw);
        hp = lds.hp;
        qp = lds.qp;
        npairs = k * (k - 1) / 2;
        all = (1u << k) - 1u;
        info = reinterpret_cast<uint32_t*>(sm + lds.info_off);
        set_order = reinterpret_cast<uint16_t*>(sm + lds.order_off);
        P = reinterpret_cast<double*>(sm + lds.P_off);
        t_s = reinterpret_cast<float*>(sm + lds.t_off);
        B_s = reinterpret_cast<float*>(sm + lds.B_off);
        M_s = reinterpret_cast<float*>(sm + lds.M_off);
        hi_s = sm + lds.hi_off;
        lo_s = sm + lds.lo_off;
        q16 = reinterpret_cast<uint16_t*>(sm + lds.q_off);
        scratch = sm + lds.run_off;
        raw = is_raw;
        prep = raw ? nullptr : task.prepared + (size_t)inst * task.y.stride;
        slot = task.slots + (size_t)blockIdx.x * task.slot_dwords;
        // valid once the ranges are known: the run minima of a wave, and the rows behind those if they fit
        rd = (int)(__builtin_amdgcn_readfirstlane((int)sh.widest) + 1) / 2;
        const uint32_t over16 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.over16);
        const uint32_t over32 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.over32);
        const uint32_t over64 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.over64);
        const uint32_t run_pitch = over64 ? run_dwords(1) : over32 ? run_dwords(2) : over16 ? run_dwords(4) : run_dwords(8);
        run32 = reinterpret_cast<uint32_t*>(sm + lds.run_off) + (uint32_t)wave * run_pitch;
        const uint32_t runs_end = lds.run_off + (uint32_t)waves * run_pitch * 4u;
        query = reinterpret_cast<uint32_t*>(sm + runs_end);
        const uint32_t row_off = runs_end + (__builtin_amdgcn_readfirstlane((int)sh.whole) ? query_bytes(L, k) : 0u);
        lds_rows = reinterpret_cast<uint32_t*>(sm + row_off);
        in_lds = may_use_lds && row_off + row_dwords(k, rd) * 4u <= task.lds_bytes;
    }
    __device__ __forceinline__ BandsCtx ctx() const {
        return BandsCtx{reinterpret_cast<const uint32_t*>(q16), hi_s, info, nullptr, L, k, rd, hp, qp};
    }
};
#define PPO_BANDS_VIEW                                                                                                    \
    const BandsView view(sm, task, inst, RAW, PART == kWhole);                                                \
    [[maybe_unused]] const int tid = view.tid, lane = view.lane, wave = view.wave, waves = view.waves, threads = view.threads; \
    [[maybe_unused]] const int L = view.L, k = view.k, hp = view.hp, qp = view.qp, npairs = view.npairs, rd = view.rd;     \
    [[maybe_unused]] const uint32_t all = view.all;                                                                        \
    [[maybe_unused]] BandsShared& sh = view.sh;                                                                           \
    [[maybe_unused]] uint32_t *info = view.info, *lds_rows = view.lds_rows, *slot = view.slot, *run32 = view.run32;        \
    [[maybe_unused]] uint32_t* query = view.query;                                                                        \
    [[maybe_unused]] uint16_t *set_order = view.set_order, *q16 = view.q16;                                                \
    [[maybe_unused]] double* P = view.P;                                                                                   \
    [[maybe_unused]] float *t_s = view.t_s, *B_s = view.B_s, *M_s = view.M_s;                                              \
    [[maybe_unused]] unsigned char *hi_s = view.hi_s, *lo_s = view.lo_s, *scratch = view.scratch;                          \
    [[maybe_unused]] constexpr bool raw = RAW;                                                                             \
    [[maybe_unused]] const bool in_lds = view.in_lds;                                                      \
    [[maybe_unused]] const unsigned char* prep = view.prep;

// The sets' rows and places, requested by the kernel before anything else.
template <int KMAX>
struct BandsFirst {
    static constexpr int kEach = KMAX <= kSmallK ? 1 : (1 << PPO_MAX_K) / (kSubsetMaxWaves * 64);   // 2^k threads, or 1024
    uint32_t value[kEach], level;
};

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_inputs(unsigned char* sm, const BandsTask& task, uint32_t inst, bool fresh,
                                              const BandsFirst<KMAX>& sets) {
    PPO_BANDS_VIEW
    if (raw) {
        // inputs, all requested before the first is waited for (a workgroup has a thread for every element); a transfer
        // size of zero is +0 whatever its sign bit says
        float* m_s = reinterpret_cast<float*>(scratch);
        const int a = tid / k, b = tid - a * k;   // the element with the smaller row index is the one read
        float tv = 0.0f, mv = 0.0f, Mv = 0.0f, Bv = 0.0f;
        if (tid < L) {
            tv = task.t[(size_t)inst * L + tid];
            mv = task.m[(size_t)inst * L + tid];
        }
        if (tid < k * k) Bv = task.B[(size_t)inst * k * k + (a < b ? tid : b * k + a)];
        if (tid < k) Mv = task.M[(size_t)inst * k + tid];
        if (tid < L) {
            t_s[tid] = tv == 0.0f ? 0.0f : tv;
            m_s[tid] = mv;
        }
        if (tid < k * k) B_s[tid] = Bv;
        if (tid < k) M_s[tid] = Mv;
        if (fresh && tid <= k + 1) sh.level[tid] = sets.level;
    } else {
        if (fresh && tid <= k + 1) sh.level[tid] = sets.level;
        for (int i = tid; i < k * (L + 1); i += threads) {
            const int j = i / (L + 1);
            lo_s[j * hp + i - j * (L + 1)] = prep[task.y.lo_off + i];
        }
    }
    if (tid == 0) {
        sh.over16 = sh.over32 = sh.over64 = 0u;
        sh.widest = 1u;
        sh.whole = sh.longest = 0u;
        sh.lo_bits = sh.hi_bits = 0u;
    }
}

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_prefix(unsigned char* sm, const BandsTask& task, uint32_t inst, bool fresh,
                                              const BandsFirst<KMAX>& sets) {
    PPO_BANDS_VIEW
    if (fresh) {
#pragma unroll
        for (int i = 0; i < BandsFirst<KMAX>::kEach; ++i) {
            const uint32_t set = (uint32_t)(tid + i * threads);
            if (set <= all) {
                set_order[sh.level[__popc(set)] + (sets.value[i] >> 16)] = (uint16_t)set;   // in the order of the levels
                info[set] = sets.value[i] & 0xFFFFu;
            }
        }
    }
    if (raw) {
        const float* m_s = reinterpret_cast<const float*>(scratch);
        if (wave == 0) {
            // prefix sums in index order in binary64 (the definition fixes the order)
            // (a lane's weight is fetched from its register: no memory access in the chain of additions; all lanes add
            // and store the same: a store by one lane took 4096 x (96, 8) from 612 to 634 us)
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
            // (patterns of values >= 0 are in the order of the values)
            tmin = __uint_as_float(wave_min(__float_as_uint(tmin)));
            tmax = __uint_as_float(wave_max(__float_as_uint(tmax)));
            bmin = __uint_as_float(wave_min(__float_as_uint(bmin)));
            bmax = __uint_as_float(wave_max(__float_as_uint(bmax)));
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
    }
}

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_windows(unsigned char* sm, const BandsTask& task, uint32_t inst) {
    PPO_BANDS_VIEW
    // hi[j][e] does not shrink as e grows (sums of weights >= 0), so a binary search finds what a scan would
    {
        const int chunks = (L + 64) >> 6;   // of 64 cuts 0 .. L, for a wave
        for (int item = wave; item < k * chunks; item += waves) {
            const int j = item / chunks, e = (item - j * chunks) * 64 + lane;
            if (e > L) continue;
            int end = e;
            if (RAW) {
                const double cap = (double)M_s[j], at = P[e];
                int step = 1;
                while (step < L) step <<= 1;
                for (; step >= 1; step >>= 1) {
                    const int e2 = end + step;
                    if (e2 <= L && P[e2] - at <= cap) end = e2;
                }
            } else {
                int top = L;   // last end whose window starts at or before e
                while (end < top) {
                    const int mid = (end + top + 1) >> 1;
                    if (lo_s[j * hp + mid] <= e) end = mid; else top = mid - 1;
                }
            }
            hi_s[j * hp + e] = (unsigned char)end;
        }
    }
}

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_ranges(unsigned char* sm, const BandsTask& task, uint32_t inst) {
    PPO_BANDS_VIEW
    // Ranges of the sets: from the capacities together (a little wider than the sets need, by up to a layer and a half a
    // node, but without a chain of levels: 0.6 us against 3.7 with 8 nodes), or where these are not at hand
    // level by level from the windows.
    unsigned char* first = scratch;
    unsigned char* last = scratch + (1u << k);
    if (!raw) {
        __syncthreads();
        if (tid == 0) {
            first[0] = 0;
            last[0] = (unsigned char)L;
        }
        for (int c = 1; c <= k; ++c) {
            __syncthreads();
            const uint32_t from = sh.level[c], count = sh.level[c + 1] - from;
            for (uint32_t i = (uint32_t)tid; i < 2u * count; i += (uint32_t)threads) {
                const bool back = i >= count;
                const uint32_t set = set_order[from + (back ? i - count : i)];
                const unsigned char* of = back ? last : first;
                const unsigned char* window = back ? lo_s : hi_s;
                int x = back ? L : 0;
                // four members at a time, so that their reads are in flight together (twice the same one does no harm)
                for (uint32_t bits = set; bits;) {
                    int j[4], at[4], y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        j[u] = bits ? __ffs(bits) - 1 : j[u > 0 ? u - 1 : 0];
                        bits &= bits - 1u;
                        at[u] = of[set & ~(1u << j[u])];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[u] = window[j[u] * hp + at[u]];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x = back ? (y[u] < x ? y[u] : x) : (y[u] > x ? y[u] : x);
                }
                (back ? last : first)[set] = (unsigned char)x;
            }
        }
        __syncthreads();
    }
    {
        uint32_t flags = 0, widest = 0;   // over 16 from bit 0, over 32 from bit 16; over 64 apart
        uint32_t flags64 = 0;
        for (uint32_t set = (uint32_t)tid; set <= all; set += (uint32_t)threads) {
            const int c = __popc(set);
            int a, b;
            if (raw) {
                // Segments that fit one by one fit together, up to the rounding of the differences and sums.
                double in = 0.0, out = 0.0;
#pragma unroll
                for (int j = 0; j < KMAX; ++j) {
                    if (j >= k) break;
                    const double cap = (double)M_s[j];
                    const bool member = (set >> j) & 1u;
                    in += member ? cap : 0.0;
                    out += member ? 0.0 : cap;
                }
                in *= 1.0 + 1e-13;
                out *= 1.0 + 1e-13;
                const double whole = P[L];
                int step = 1;
                a = L;
                b = 0;
                while (step < L) step <<= 1;
                for (; step >= 1; step >>= 1) {   // two searches side by side
                    const int e2 = b + step, e3 = a - step;
                    const double p2 = P[e2 <= L ? e2 : L], p3 = P[e3 >= 0 ? e3 : 0];
                    if (e2 <= L && p2 <= out) b = e2;
                    if (e3 >= 0 && whole - p3 <= in) a = e3;
                }
            } else {
                a = last[set];
                b = first[all ^ set];
            }
            a = a > k - c ? a : k - c;
            b = b < L - c ? b : L - c;
            uint32_t x = info[set] & 0x7FFFu;
            if (a > b || c == 0) {
                x |= kEmptySet;
            } else {
                const int base = a & ~1, width = b - base + 1;
                x = make_info(x, base, b);
                flags |= (width > 16 ? 1u << c : 0u) | (width > 32 ? 0x10000u << c : 0u);
                flags64 |= width > 64 ? 1u << c : 0u;
                widest = (uint32_t)width > widest ? (uint32_t)width : widest;
            }
            info[set] = x;
        }
        if ((uint32_t)wave * 64u <= all) {
            flags = wave_or(flags);
            flags64 = wave_or(flags64);
            widest = wave_max(widest);
            if (lane == 0) {
                atomicOr(&sh.over16, flags & 0xFFFFu);
                atomicOr(&sh.over32, flags >> 16);
                atomicOr(&sh.over64, flags64);
                atomicMax(&sh.widest, widest);
            }
        }
    }
}

// Window queries of whole rows: (e, min(hi, L-1)] is covered by two runs of 2^r entries, the one that starts at e + 1 and the
// one that ends at its end; their byte offsets in a wave's run minima, 16 bits each, as if those started at the cut 0 (they
// start at up to 12: the entries for empty windows, behind the run minima, are pointed at in their middle).
__device__ __forceinline__ void bands_queries(BandsShared& sh, const unsigned char* hi_s, uint32_t* query, int L, int k, int hp, int threads) {
    constexpr uint32_t kNone = kRunNone * 4u + 2u * (uint32_t)PPO_MAX_K;
    const int pitch = (int)query_pitch(L);
    uint32_t longest = 0;
    for (int j = (int)threadIdx.x >> 6; j < k; j += threads >> 6)
    for (int e = (int)threadIdx.x & 63; e < pitch; e += 64) {
        uint32_t d = kNone | (kNone << 16);
        const int hi = e < L ? (int)hi_s[j * hp + e] : 0, top = hi < L - 1 ? hi : L - 1;
        if (top > e) {
            const int r = 31 - __clz(top - e) < run_levels(1) - 1 ? 31 - __clz(top - e) : run_levels(1) - 1;
            d = (uint32_t)(r * 256 + (e + 1) * 2) | (uint32_t)(r * 256 + (top - (1 << r) + 1) * 2) << 16;
            longest = (uint32_t)r > longest ? (uint32_t)r : longest;
        }
        query[j * pitch + e] = d;
    }
    longest = wave_max(longest);
    if ((threadIdx.x & 63u) == 0u) atomicMax(&sh.longest, longest);
}
static_assert((run_dwords(1) - kRunNone) * 4u >= 2u * PPO_MAX_K + 2u && PPO_MAX_L == 128, "entries for empty windows, and the runs of a row");

// Whether an instance's rows are better worked as long as they can be.  Ranges of more than 64 entries take a set to a wave, and a
// row by bands_level is then longer than one whose windows are looked up in a table: 75 vector instructions, for up to eight
// sets at a time, against 47.  In the staged search whole rows have to win by a fifth (narrow ones may fit LDS), and by a half
// where the levels are launches of their own, each of which makes the table (one search of 100 layers on 11 nodes: 83 us by
// ranges, 91 so).
// Ample memory, in us without ranges / with them / so: 4096 x (96, 8) of random chains with four times what they need 1067 / 1483 /
// 1104, with twice 994 / 1467 / 1037; 1024 x (80, 7) 157 / 215 / 156; staged 300 x (100, 10) 422 / 566 / 416.
template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_whole_rows(unsigned char* sm, const BandsTask& task, uint32_t inst) {
    PPO_BANDS_VIEW
    const uint32_t over16 = sh.over16, over32 = sh.over32, over64 = sh.over64;
    uint32_t by_range = 0, by_rows = 0;   // vector instructions
    for (int C = 1; C < k; ++C) {
        const uint32_t here = 3u << C, count = (sh.level[C + 1] - sh.level[C]) * (uint32_t)(k - C);
        by_range += count * (over64 & here ? 75u : over32 & here ? 38u : over16 & here ? 19u : 10u);
        by_rows += count * 47u;
    }
    if (10u * by_range <= (RAW ? 10u : PART == kHead ? 15u : 12u) * by_rows || (PART == kHead && !task.query_bytes)) return;
    __syncthreads();
    // a range is all cuts that leave a layer to every node
    for (uint32_t set = (uint32_t)tid; set <= all; set += (uint32_t)threads) {
        const int c = __popc(set);
        info[set] = c ? make_info(info_row(info[set]), whole_base(k, c), L - c) : info_row(info[set]) | kEmptySet;
    }
    if (tid == 0) {
        sh.whole = 1u;
        sh.over64 = ~0u;
        sh.widest = (uint32_t)(k > 1 ? L - k + 2 : L);
    }
    bands_queries(sh, hi_s, query, L, k, hp, threads);
    __syncthreads();
}

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_codes(unsigned char* sm, const BandsTask& task, uint32_t inst) {
    PPO_BANDS_VIEW
    const uint32_t lo_bits = sh.lo_bits, hi_bits = sh.hi_bits;
    // quotients of every ordered pair of nodes (Eq. 3): entry e is that of the cut e; +inf where there is none and
    // from a node to itself (pair npairs + j)
    const uint32_t span = hi_bits - lo_bits;
    const int shift = span < kFinestCodes ? 0 : 32 - __clz(span / kFinestCodes);
    for (int p = wave; p < npairs + k; p += waves) {
        int a = p - npairs, b = a;
        if (p < npairs) pair_nodes(p, k, a, b);
        const float bw = B_s[a * k + b];
        for (int e = lane; e < 2 * qp; e += 64) {
            uint32_t c = kCodeInf;
            if (a != b && e >= 1 && e < L) {
                if (raw) {
                    const uint32_t bits = __float_as_uint(__fdiv_rn(t_s[e - 1], bw));
                    if (bits == 0u || bits < lo_bits) c = kCodeZero;
                    else if (bits <= hi_bits) c = kCodeZero + 1u + ((bits - lo_bits) >> shift);
                } else {
                    c = reinterpret_cast<const uint16_t*>(prep + task.y.qc_off)[p * L + e - 1];
                }
            }
            put_code(q16, k, qp, a, b, e, c);
        }
    }
}

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_singles(unsigned char* sm, const BandsTask& task, uint32_t inst) {
    PPO_BANDS_VIEW
    // sets of one node: its segment runs to the end of the chain
    for (int idx = tid; idx < k * rd; idx += threads) {
        const int j = idx / rd, d = idx - j * rd;
        const uint32_t x = info[1u << j];
        const int e = info_base(x) + 2 * d;
        const uint32_t v0 = e < L && hi_s[j * hp + e] == L ? kCodeZero : kCodeInf;
        const uint32_t v1 = e + 1 < L && hi_s[j * hp + e + 1] == L ? kCodeZero : kCodeInf;
        const uint32_t at = info_row(x) * (uint32_t)rd + (uint32_t)d;
        if (in_lds) lds_rows[at] = v0 | (v1 << 16);
        else slot[at] = v0 | (v1 << 16);
    }
    if (tid == 0) {
        sh.bucket_lo = ~0u;
        sh.bucket_hi = 0u;
    }
}

template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_levels(unsigned char* sm, const BandsTask& task, uint32_t inst, int from, int to) {
#define PPO_BANDS_LEVEL(C_)                                                                                            \
    if (C_ < KMAX && C_ >= from && C_ <= to) {                                                                          \
        {                                                                                                               \
            PPO_BANDS_VIEW                                                                                             \
            if (in_lds) bands_level_any<C_>(sh, view.ctx(), set_order, lane, wave, waves, task, query, run32, lds_rows); \
            else bands_level_any<C_>(sh, view.ctx(), set_order, lane, wave, waves, task, query, run32, slot);          \
        }                                                                                                               \
        __syncthreads();                                                                                                \
    }
    PPO_BANDS_LEVEL(1)
    PPO_BANDS_LEVEL(2)
    PPO_BANDS_LEVEL(3)
    PPO_BANDS_LEVEL(4)
    PPO_BANDS_LEVEL(5)
    PPO_BANDS_LEVEL(6)
    PPO_BANDS_LEVEL(7)
    PPO_BANDS_LEVEL(8)
    PPO_BANDS_LEVEL(9)
    PPO_BANDS_LEVEL(10)
    PPO_BANDS_LEVEL(11)
#undef PPO_BANDS_LEVEL
}

// The least entry of the full set's rows (the last k ones; their range is the cut 0 alone); kCodeInf: none.
template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ uint32_t bands_best(unsigned char* sm, const BandsTask& task, uint32_t inst) {
    PPO_BANDS_VIEW
    uint32_t best = kCodeInf;
    if (lane < k && !(info[all] & kEmptySet)) {
        const uint32_t at = (info_row(info[all]) + (uint32_t)lane) * (uint32_t)rd;
        best = (in_lds ? lds_rows[at] : slot[at]) & 0xFFFFu;
    }
    return wave_min(best);
}

// Range of the quotients with the code `best`.
template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_bucket(unsigned char* sm, const BandsTask& task, uint32_t inst, uint32_t best) {
    PPO_BANDS_VIEW
    uint32_t least = ~0u, most = 0u;
    for (int p = wave; p < npairs; p += waves) {
        int a, b;
        pair_nodes(p, k, a, b);
        for (int i = lane; i < L - 1; i += 64)
            if (q16[(a * k + b) * (2 * qp) + i + 1] == best) {
                const uint32_t bits = __float_as_uint(__fdiv_rn(t_s[i], B_s[a * k + b]));
                least = bits < least ? bits : least;
                most = bits > most ? bits : most;
            }
    }
    least = wave_min(least);
    most = wave_max(most);
    if (lane == 0 && least != ~0u) {
        atomicMin(&sh.bucket_lo, least);
        atomicMax(&sh.bucket_hi, most);
    }
}

// The lexicographically smallest optimal ordering, position by position: F = cuts that the chosen prefix reaches with all
// its links at most beta*.  A candidate completes to an optimum iff A[unused][j][e] <= beta* for some e in F whose link into
// it is at most beta*; the smallest such node is taken (G = those e: other starts lead to no cut of an optimum), and F for
// the next position is the set of cuts that a window of that node starting in G covers (hi[j][.] does not decrease, so the
// latest start below a cut decides).  F and G by entries of the unused set's rows; a wave per candidate, then every wave takes
// the same step (walked by one wave, four candidates at a time, a position took 1.4 us, three times as long).
template <int KMAX, int PART, bool RAW, bool WIDE>
__device__ __forceinline__ void bands_trace(unsigned char* sm, const BandsTask& task, uint32_t inst, uint32_t best,
                                             uint32_t best_bits) {
    PPO_BANDS_VIEW
    unsigned long long* cand = reinterpret_cast<unsigned long long*>(scratch);   // [2][k][2], the two halves in turns
    unsigned long long F0 = 1ull, F1 = 0ull;   // the first segment starts at 0
    unsigned long long my_start0 = 0ull, my_start1 = 0ull;   // lane s: G of the node at position s
    uint32_t unused = all, rank = 0, x = (uint32_t)__builtin_amdgcn_readfirstlane((int)info[all]);
    int prev = 0, my_node = 0, my_base = 0;
    for (int s = 0; s < k; ++s) {
        const int base = info_base(x), width = info_end(x) - base + 1;
        const int i0 = lane < width ? lane : 0, i1 = WIDE && lane + 64 < width ? lane + 64 : 0;
        unsigned long long* buf = cand + (s & 1) * 2 * k;
        for (int j = wave; j < k; j += waves) {
            unsigned long long g0 = 0ull, g1 = 0ull;
            if ((unused >> j) & 1u) {
                const uint32_t at = mul24(info_row(x) + (uint32_t)__popc(unused & ((1u << j) - 1u)), (uint32_t)(2 * rd));
                const uint16_t* link = q16 + (prev * k + j) * (2 * qp) + base;
                const uint16_t* row = (in_lds ? reinterpret_cast<const uint16_t*>(lds_rows) : reinterpret_cast<const uint16_t*>(slot)) + at;
                const uint32_t a0 = in_lds ? reinterpret_cast<const uint16_t*>(lds_rows)[at + i0] : reinterpret_cast<const uint16_t*>(slot)[at + i0];
                const uint32_t q0 = s == 0 ? 0u : link[i0];   // beyond the first position F holds no cut 0
                g0 = __ballot(((F0 >> lane) & 1ull) && a0 <= best && q0 <= best);
                if (WIDE) {
                    const uint32_t q1 = s == 0 ? 0u : link[i1];
                    g1 = __ballot(((F1 >> lane) & 1ull) && row[i1] <= best && q1 <= best);
                }
            }
            if (lane == 0) {
                buf[2 * j] = g0;
                if (WIDE) buf[2 * j + 1] = g1;
            }
        }
        __syncthreads();
        const unsigned long long c0 = lane < k ? buf[2 * lane] : 0ull, c1 = WIDE && lane < k ? buf[2 * lane + 1] : 0ull;
        const unsigned long long ok = __ballot((c0 | c1) != 0ull);   // (some completion of the prefix reaches the optimum)
        const int chosen = ok ? __ffsll((long long)ok) - 1 : __ffs(unused) - 1;
        auto of_lane = [&](unsigned long long v) -> unsigned long long {
            return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, chosen) |
                   ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), chosen) << 32);
        };
        const unsigned long long G0 = of_lane(c0), G1 = WIDE ? of_lane(c1) : 0ull;
        if (lane == s) {
            my_node = chosen;
            my_base = base;
            my_start0 = G0;
            my_start1 = G1;
        }
        const uint32_t below = unused & ((1u << chosen) - 1u);
        rank = rank * (uint32_t)(k - s) + (uint32_t)__popc(below);   // the rank's digit in the factorial system
        unused &= ~(1u << chosen);
        prev = chosen;
        if (s == k - 1) break;
        x = (uint32_t)__builtin_amdgcn_readfirstlane((int)info[unused]);
        const int base2 = info_base(x), width2 = x & kEmptySet ? 0 : info_end(x) - base2 + 1;
        const unsigned char* window = hi_s + chosen * hp + base;
        auto covered = [&](int i) -> bool {
            const int upto = base2 + i - base;   // entries of G before the cut
            int from = -1;
            if (WIDE && upto > 64) {
                const unsigned long long m = upto >= 128 ? G1 : G1 & ((1ull << (upto - 64)) - 1ull);
                if (m) from = 127 - __clzll((long long)m);
            }
            if (!WIDE || from < 0) {
                const int u = upto < 64 ? upto : 64;
                const unsigned long long m = u > 0 ? G0 << ((64 - u) & 63) : 0ull;   // the last of them on top
                from = m ? u - 1 - __clzll((long long)m) : -1;
            }
            return i < width2 && from >= 0 && (int)window[from < 0 ? 0 : from] >= base2 + i;
        };
        F0 = __ballot(covered(lane));
        if (WIDE) F1 = __ballot(covered(lane + 64));
    }
    if (wave != 0) return;
    if (!RAW) {
        if (lane == 0) task.key[inst] = ((unsigned long long)best_bits << 32) | rank;
        return;
    }
    // cuts, latest segment first: each time the smallest start (reached by the prefix, link at most beta*) whose window
    // covers the end
    int e = L, my_cut = 0;
    for (int s = k - 1; s >= 1; --s) {
        const int js = __builtin_amdgcn_readlane(my_node, s), base = __builtin_amdgcn_readlane(my_base, s);
        auto start_of = [&](unsigned long long v) -> unsigned long long {
            return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, s) |
                   ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), s) << 32);
        };
        const int e0 = base + lane, e1 = e0 + 64;
        const unsigned long long m0 = __ballot(((start_of(my_start0) >> lane) & 1ull) && e0 < e && hi_s[js * hp + (e0 < L ? e0 : L)] >= e);
        unsigned long long m1 = 0ull;
        if (WIDE) m1 = __ballot(((start_of(my_start1) >> lane) & 1ull) && e1 < e && hi_s[js * hp + (e1 < L ? e1 : L)] >= e);
        e = base + (m0 ? __ffsll((long long)m0) - 1 : 63 + __ffsll((long long)m1));
        if (lane == s - 1) my_cut = e;
    }
    if (lane == 0) task.beta[inst] = __uint_as_float(best_bits);
    if (lane < k) task.order[(size_t)inst * k + lane] = my_node;
    if (lane < k - 1) task.cuts[(size_t)inst * (k - 1) + lane] = my_cut;
}

// No ordering is feasible.
template <int KMAX, int PART, bool RAW>
__device__ __forceinline__ void bands_infeasible(const BandsTask& task, uint32_t inst) {
    const int tid = threadIdx.x, k = task.k;
    if (!RAW) {
        if (tid == 0) task.key[inst] = (unsigned long long)kInfBits << 32;
        return;
    }
    if (tid == 0) task.beta[inst] = __uint_as_float(kInfBits);
    if (tid < k) task.order[(size_t)inst * k + tid] = -1;
    if (tid < k - 1) task.cuts[(size_t)inst * (k - 1) + tid] = -1;
}

template <int KMAX, int PART, bool RAW>
__global__ __launch_bounds__(kSubsetMaxWaves * 64, KMAX <= kSmallK ? 8 : 4) void bands_solve_kernel(const BandsTask task) {
    extern __shared__ __align__(16) unsigned char sm[];
    BandsFirst<KMAX> sets;
    bool fresh = PART != kTail;
    if (fresh) {
        const uint32_t all = (1u << task.k) - 1u;
#pragma unroll
        for (int i = 0; i < BandsFirst<KMAX>::kEach; ++i) {
            const uint32_t set = threadIdx.x + (uint32_t)i * blockDim.x;
            sets.value[i] = set <= all ? kSetValues.row_and_place[set] : 0u;
        }
        sets.level = (int)threadIdx.x <= task.k + 1 ? kSetValues.level[task.k][threadIdx.x] : 0u;
    }
    for (uint32_t inst = blockIdx.x; inst < (uint32_t)task.n_inst; inst += gridDim.x) {
        if (PART == kTail) {
            const BandsLds lds = BandsLds::make(task.L, task.k, false);
            const uint4* image = reinterpret_cast<const uint4*>(task.slots + (size_t)blockIdx.x * task.slot_dwords + area_dwords(task.k, task.L));
            for (uint32_t i = threadIdx.x; i < lds.run_off / 16u; i += blockDim.x) reinterpret_cast<uint4*>(sm)[i] = image[i];
        } else {
            bands_inputs<KMAX, PART, RAW>(sm, task, inst, fresh, sets);
            __syncthreads();
            bands_prefix<KMAX, PART, RAW>(sm, task, inst, fresh, sets);
            fresh = false;
            __syncthreads();
            bands_windows<KMAX, PART, RAW>(sm, task, inst);
            bands_ranges<KMAX, PART, RAW>(sm, task, inst);
            bands_codes<KMAX, PART, RAW>(sm, task, inst);
        }
        __syncthreads();
        if (reinterpret_cast<const BandsShared*>(sm)->over64) {   // (the same in all threads: nobody clears it)
            if (PART != kTail) {
                bands_whole_rows<KMAX, PART, RAW>(sm, task, inst);
            } else if (reinterpret_cast<const BandsShared*>(sm)->whole) {
                PPO_BANDS_VIEW
                bands_queries(sh, view.hi_s, query, L, k, hp, threads);
            }
        }
        if (PART != kTail) bands_singles<KMAX, PART, RAW>(sm, task, inst);
        else if (threadIdx.x == 0) {
            BandsShared& sh = *reinterpret_cast<BandsShared*>(sm);
            sh.bucket_lo = ~0u;
            sh.bucket_hi = 0u;
        }
        __syncthreads();
        if (PART == kHead) {
            bands_levels<KMAX, PART, RAW>(sm, task, inst, 1, task.from);
            const BandsLds lds = BandsLds::make(task.L, task.k, false);
            uint4* image = reinterpret_cast<uint4*>(task.slots + (size_t)blockIdx.x * task.slot_dwords + area_dwords(task.k, task.L));
            for (uint32_t i = threadIdx.x; i < lds.run_off / 16u; i += blockDim.x) image[i] = reinterpret_cast<const uint4*>(sm)[i];
            __syncthreads();
            continue;
        }
        uint32_t best, best_bits = kInfBits;
        for (int from = PART == kTail ? task.to : 1;; from = 1) {
            bands_levels<KMAX, PART, RAW>(sm, task, inst, from, task.k - 1);
            best = bands_best<KMAX, PART, RAW>(sm, task, inst);
            if (best >= kCodeInf) break;
            if (!RAW) {   // its codes are exact
                const float* dec = reinterpret_cast<const float*>(task.prepared + (size_t)inst * task.y.stride + task.y.dec_off);
                best_bits = __float_as_uint(dec[best - kCodeZero]);
                break;
            }
            if (best == kCodeZero) {   // the optimum is 0 (after the first pass it lies in the range)
                best_bits = 0u;
                break;
            }
            bands_bucket<KMAX, PART, RAW>(sm, task, inst, best);
            __syncthreads();
            BandsShared& sh = *reinterpret_cast<BandsShared*>(sm);
            const uint32_t low = sh.bucket_lo, high = sh.bucket_hi;
            if (low >= high) {
                best_bits = low;
                break;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                sh.lo_bits = low;
                sh.hi_bits = high;
            }
            __syncthreads();
            bands_codes<KMAX, PART, RAW>(sm, task, inst);
            bands_singles<KMAX, PART, RAW>(sm, task, inst);
            __syncthreads();
        }
        if (best >= kCodeInf || best_bits >= kInfBits) bands_infeasible<KMAX, PART, RAW>(task, inst);
        else if (reinterpret_cast<const BandsShared*>(sm)->widest > 64u) bands_trace<KMAX, PART, RAW, true>(sm, task, inst, best, best_bits);
        else bands_trace<KMAX, PART, RAW, false>(sm, task, inst, best, best_bits);
        __syncthreads();   // the next instance overwrites what the last steps read
    }
}
#undef PPO_BANDS_VIEW

// One level of the sets over many workgroups: grid.x of them per instance, grid.y = instance.
constexpr int kLevelWaves = 8;
template <int C>
__global__ __launch_bounds__(kLevelWaves * 64, 6) void bands_level_kernel(const BandsTask task) {
    extern __shared__ __align__(16) unsigned char sm[];
    const int L = task.L, k = task.k;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const BandsLds lds = BandsLds::make(L, k, false);
    uint32_t* slot = task.slots + (size_t)blockIdx.y * task.slot_dwords;
    const unsigned char* image = reinterpret_cast<const unsigned char*>(slot + area_dwords(k, L));
    const BandsShared& shg = *reinterpret_cast<const BandsShared*>(image);
    {
        // four sets to a wave need fewer workgroups than the grid has room for
        const uint32_t here = 3u << C, nsets = shg.level[C + 1] - shg.level[C];
        const int s = (int)(task.splits >> (4 * C));
        const uint32_t G = shg.over64 & here ? 1u : shg.over32 & here ? 2u : shg.over16 & here ? 4u : 8u;
        const uint32_t items = shg.whole ? nsets << ((task.whole_splits >> (2 * C)) & 3u) : ((nsets + G - 1u) / G) << (G >= 4u ? (s >> 2) & 3 : s & 3);
        if (blockIdx.x * (uint32_t)kLevelWaves >= items) return;
    }
    // the header, the sets and the window ends, and the quotients; the rest of the image is not needed
    for (uint32_t i = (uint32_t)tid; i < lds.P_off / 16u; i += blockDim.x) reinterpret_cast<uint4*>(sm)[i] = reinterpret_cast<const uint4*>(image)[i];
    const uint32_t hi_bytes = lds.lo_off - lds.hi_off;
    for (uint32_t i = (uint32_t)tid; i < hi_bytes / 16u; i += blockDim.x)
        reinterpret_cast<uint4*>(sm + lds.hi_off)[i] = reinterpret_cast<const uint4*>(image + lds.hi_off)[i];
    for (uint32_t i = (uint32_t)tid; i < (lds.run_off - lds.q_off) / 16u; i += blockDim.x)
        reinterpret_cast<uint4*>(sm + lds.q_off)[i] = reinterpret_cast<const uint4*>(image + lds.q_off)[i];
    __syncthreads();
    BandsShared& sh = *reinterpret_cast<BandsShared*>(sm);
    uint32_t* run32 = reinterpret_cast<uint32_t*>(sm + lds.run_off) + (uint32_t)wave * run_dwords(1);
    uint32_t* query = reinterpret_cast<uint32_t*>(sm + lds.run_off) + (uint32_t)kLevelWaves * run_dwords(1);
    if (sh.whole) {
        bands_queries(sh, sm + lds.hi_off, query, L, k, lds.hp, (int)blockDim.x);
        __syncthreads();
    }
    const BandsCtx ctx{reinterpret_cast<const uint32_t*>(sm + lds.q_off), sm + lds.hi_off,
                        reinterpret_cast<const uint32_t*>(sm + lds.info_off), nullptr, L, k, ((int)sh.widest + 1) / 2, lds.hp, lds.qp};
    bands_level_any<C>(sh, ctx, reinterpret_cast<const uint16_t*>(sm + lds.order_off), lane, (int)blockIdx.x * kLevelWaves + wave,
                        (int)gridDim.x * kLevelWaves, task, query, run32, slot);
}

namespace {
constexpr size_t kLdsGrain = 1280;   // a workgroup's LDS is a multiple of it
// (A search of few instances, or of ample memory on whole rows, wants all the waves there are: 16 x (100, 8) with three times the
// memory they need 85 us staged with eight, 65 with sixteen.)
// Eight waves: with four, ranges that are not narrow take rows in global memory (2048 x (96, 8) of random chains 402 us, with
// eight 327); with sixteen the phases that one wave works alone leave more idle (4096 x (96, 8) of transformers 480 us against 360).
int bands_waves(int L, int k, int n_inst) { return k <= kSmallK && (k < 7 || L - k + 2 <= 64 || n_inst > 256) ? 8 : kSubsetMaxWaves; }

// Parts of the nodes outside a set for `waves` waves: the least number of rows that one wave works in turn.
int best_split(int sets, int outside, int waves) {
    int best = 0, least = 1 << 30;
    for (int s = 0; s < 4 && (1 << s) <= outside; ++s) {
        const int per = (outside + (1 << s) - 1) >> s, rounds = ((sets << s) + waves - 1) / waves;
        const int cost = rounds * (2 * per + 1);   // loading the rows of the sets costs about half a row's work
        if (cost < least) {
            least = cost;
            best = s;
        }
    }
    return best;
}
int level_cost(int k, int C, int waves) {   // rows that one wave works in turn, with two sets to a wave
    const int sets = ((int)kSetsHost.choose[k][C] + 1) / 2, s = best_split(sets, k - C, waves);
    return (((sets << s) + waves - 1) / waves) * ((k - C + (1 << s) - 1) >> s);
}
void set_splits(BandsTask& task, int C, int waves) {
    const int k = task.k, n = (int)kSetsHost.choose[k][C];
    const int two = best_split((n + 1) / 2, k - C, waves), four = best_split((n + 3) / 4, k - C, waves);
    task.splits |= (unsigned long long)(two | (four << 2)) << (4 * C);
    task.whole_splits |= (uint32_t)best_split(n, k - C, waves) << (2 * C);
}
void set_splits(BandsTask& task, int waves) {
    for (int C = 1; C < task.k; ++C) set_splits(task, C, waves);
}

// LDS of a workgroup that does the whole search, without rows; with rows as long as a range can be; and what it is given where
// there are row areas in global memory as well: a quarter of a compute unit's, for rows of narrow ranges.
uint32_t fixed_lds(int L, int k, int waves, bool raw) { return BandsLds::make(L, k, raw).run_off + (uint32_t)waves * run_dwords(L <= 64 ? 2 : 1) * 4u + query_bytes(L, k); }
size_t longest_lds(int L, int k, int waves, bool raw) { return fixed_lds(L, k, waves, raw) + (size_t)area_dwords(k, L) * 4; }
uint32_t whole_lds(int L, int k, int waves, bool raw) {
    const uint32_t fixed = fixed_lds(L, k, waves, raw), quarter = (uint32_t)kLdsBytesPerCU / 4u;
    const size_t need = longest_lds(L, k, waves, raw);
    return need <= quarter ? (uint32_t)need : fixed > quarter ? fixed : quarter;
}

size_t level_lds(int L, int k) { return BandsLds::make(L, k, false).run_off + (size_t)kLevelWaves * run_dwords(1) * 4; }
// Room for the table of whole rows where a compute unit holds as many workgroups with it (up to three: their registers).
uint32_t level_query_bytes(int L, int k) {
    auto held = [](size_t lds) { return (size_t)kLdsBytesPerCU / align_up(lds, kLdsGrain); };
    const size_t without = held(level_lds(L, k)), with = held(level_lds(L, k) + query_bytes(L, k));
    return with >= (without < 3 ? without : 3) ? query_bytes(L, k) : 0u;
}

// Launches of the levels from task.from to `last` of `cnt` instances whose tables are in place.
template <int C>
hipError_t launch_levels(const BandsTask& task, int cnt, int last, hipStream_t stream) {
    if constexpr (C < PPO_MAX_K) {
        if (C > last) return hipSuccess;
        if (C >= task.from) {
            static std::atomic<uint64_t> lds_allowed{0};
            hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&bands_level_kernel<C>), lds_allowed);
            if (e != hipSuccess) return e;
            const size_t lds = level_lds(task.L, task.k) + task.query_bytes;
            const uint32_t cap = (768u + (uint32_t)cnt - 1u) / (uint32_t)cnt;
            // nodes outside a set in as many parts as keep the workgroups that stay resident busy
            BandsTask one = task;
            one.splits = one.whole_splits = 0;
            set_splits(one, C, (int)cap * kLevelWaves);
            const int two = (int)(one.splits >> (4 * C)) & 3, whole = (int)(one.whole_splits >> (2 * C)) & 3;
            const uint32_t most = ((kSetsHost.choose[task.k][C] << (two > whole ? two : whole)) + (uint32_t)kLevelWaves - 1u) / (uint32_t)kLevelWaves;
            hipLaunchKernelGGL((bands_level_kernel<C>), dim3(most < cap ? most : cap, cnt), dim3(kLevelWaves * 64), lds, stream, one);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return launch_levels<C + 1>(task, cnt, last, stream);
    } else {
        return hipSuccess;
    }
}

template <typename Kernel>
hipError_t launch_solve(Kernel kernel, std::atomic<uint64_t>& lds_allowed, const BandsTask& task, uint32_t grid, int waves, hipStream_t stream) {
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(kernel), lds_allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * 64), task.lds_bytes, stream, task);
    return hipGetLastError();
}

// The whole search in one launch, up to kSmallK nodes: with row areas (slot > 0 bytes each) a workgroup to each, else one
// to an instance.
hipError_t launch_whole(BandsTask task, size_t slot, size_t slot_count, hipStream_t stream) {
    static std::atomic<uint64_t> allowed[2];
    const int waves = bands_waves(task.L, task.k, task.n_inst);
    auto launch = [&](uint32_t grid) -> hipError_t {
        return task.prepared ? launch_solve(&bands_solve_kernel<kSmallK, kWhole, false>, allowed[0], task, grid, waves, stream)
                             : launch_solve(&bands_solve_kernel<kSmallK, kWhole, true>, allowed[1], task, grid, waves, stream);
    };
    set_splits(task, waves);
    task.slot_dwords = (uint32_t)(slot / 4);
    if (slot != 0) {
        if (slot_count > (size_t)task.n_inst) slot_count = (size_t)task.n_inst;
        task.lds_bytes = whole_lds(task.L, task.k, waves, !task.prepared);
        return launch((uint32_t)slot_count);
    }
    task.lds_bytes = (uint32_t)longest_lds(task.L, task.k, waves, !task.prepared);
    const uint32_t each = (uint32_t)kLdsBytesPerCU / task.lds_bytes, resident = 256u * (each < 4u ? each : 4u);
    // (no more workgroups than a few times those that stay resident: a launch may have fewer than 2^32 threads)
    const uint32_t grid = (uint32_t)task.n_inst < 16u * resident ? (uint32_t)task.n_inst : 16u * resident;
    return launch(grid);
}
}  // namespace

// Whether ppo_solve goes by ranges: many instances of long chains on six to eight nodes, whose rows lie in global memory or leave
// room for three workgroups to a compute unit (six nodes: up to 80 layers).  The launch is bound by issue then,
// and rows of 20 to 60 entries in place of 65 to 128 save more than the ranges cost: in us, without and with them, 4096 x
// (96, 8) of transformers 624 / 354, of random chains 739 / 583, 1024 x (65, 8) 218 / 143, 2048 x (70, 6) 150 / 115, 4096 x (80, 6)
// 311 / 227; but 4096 x (128, 6) 286 / 298, 512 x (96, 8) 134 / 141 and 64 x (96, 8) 96 / 111: with few instances the longer
// chain of phases counts.  Ample memory (ranges as long as the chain, see bands_whole_rows) gains nothing and loses little: 4096 x
// (80, 6) 295 / 287, (128, 7) 616 / 617, (96, 8) 1067 / 1104, (112, 8) 980 / 1097, with twice the memory needed 994 / 1037 of
// (96, 8).  Up to 64 layers two sets share a wave without ranges (1024 x (50, 6): 43 / 48), up to five nodes there is little
// to share (4096 x (128, 5): 152 / 170).  With fewer areas than keep the chip busy the instances go in turns.
bool bands_apply(int L, int k, int n_inst, size_t slot, size_t slot_count) {
    return L > 64 && k >= 6 && k <= kSmallK && n_inst >= 1024 && (slot != 0 ? slot_count >= 1024 : 3u * align_up(longest_lds(L, k, 8, true), kLdsGrain) <= (size_t)kLdsBytesPerCU);
}

hipError_t launch_bands_solve(const float* t, const float* m, const float* M, const float* B, int L, int k, int n_inst,
                              float* beta_out, int32_t* cuts_out, int32_t* order_out, void* slots, size_t slot, size_t slot_count,
                              hipStream_t stream) {
    BandsTask task{};
    task.t = t;
    task.m = m;
    task.M = M;
    task.B = B;
    task.beta = beta_out;
    task.cuts = cuts_out;
    task.order = order_out;
    task.slots = static_cast<uint32_t*>(slots);
    task.L = L;
    task.k = k;
    task.n_inst = n_inst;
    return launch_whole(task, slot, slot_count, stream);
}

// Bytes of an area for one instance of the staged search by subsets; 0 if rows of the whole chain fit into LDS.
// Areas are as small as can be told beforehand: the stream-ordered allocator hands out up to 64 MiB in 60 us and more in 340 (the
// memory goes back to the system after each call that is waited for).  64 x (100, 10) takes 60 MiB; with rows of L entries it would be 65.
size_t bands_slot_bytes(int L, int k) {
    if (k <= kSmallK && longest_lds(L, k, 8, false) <= whole_lds(L, k, 8, false)) return 0;
    return (size_t)area_dwords(k, L) * 4 + (k <= kSmallK ? 0 : BandsLds::make(L, k, false).run_off);
}
int bands_resident(int k) { return k <= kSmallK ? 1024 : 256; }

// The second stage of the staged search by subsets: from the tables of ppo_prepare (window starts, exact codes) to keys.
// `slot_count` areas of bands_slot_bytes.  Beyond kSmallK nodes, and with instances for fewer workgroups than there are
// compute units, the levels that are wide enough for many workgroups are launches over all of them.
hipError_t launch_bands_keys(const Layout& y, const void* prepared, int n_inst, uint64_t* keys, void* slots, size_t slot_count,
                             hipStream_t stream) {
    BandsTask task{};
    task.prepared = static_cast<const unsigned char*>(prepared);
    task.y = y;
    task.key = reinterpret_cast<unsigned long long*>(keys);
    task.slots = static_cast<uint32_t*>(slots);
    task.L = y.L;
    task.k = y.k;
    task.n_inst = n_inst;
    const int L = y.L, k = y.k;
    const size_t slot = bands_slot_bytes(L, k);
    if (k <= kSmallK) return launch_whole(task, slot, slot_count, stream);
    static std::atomic<uint64_t> allowed[3];
    if (slot_count > (size_t)n_inst) slot_count = (size_t)n_inst;
    const BandsLds lds = BandsLds::make(L, k, false);
    task.slot_dwords = (uint32_t)(slot / 4);
    set_splits(task, kSubsetMaxWaves);
    if (slot_count >= (size_t)bands_resident(k)) {
        task.lds_bytes = (uint32_t)kLdsBytesPerCU;   // its registers leave room for one workgroup
        return launch_solve(&bands_solve_kernel<PPO_MAX_K, kWhole, false>, allowed[0], task, (uint32_t)slot_count, kSubsetMaxWaves, stream);
    }
    // levels of few sets stay with the tables and with the answer: a launch costs about as much as a dozen rows in turn
    int from = 1, to = k - 1;
    while (from < k && level_cost(k, from, kSubsetMaxWaves) <= 12) ++from;
    while (to > from && level_cost(k, to - 1, kSubsetMaxWaves) <= 12) --to;
    task.query_bytes = level_query_bytes(L, k);
    task.lds_bytes = lds.run_off + (uint32_t)kSubsetMaxWaves * run_dwords(1) * 4u + query_bytes(L, k);
    for (int first = 0; first < n_inst; first += (int)slot_count) {
        const int cnt = n_inst - first < (int)slot_count ? n_inst - first : (int)slot_count;
        BandsTask p = task;
        p.prepared += (size_t)first * y.stride;
        p.key += first;
        p.n_inst = cnt;
        p.from = from - 1;
        p.to = to;
        hipError_t e = launch_solve(&bands_solve_kernel<PPO_MAX_K, kHead, false>, allowed[1], p, (uint32_t)cnt, kSubsetMaxWaves, stream);
        if (e != hipSuccess) return e;
        BandsTask mid = p;
        mid.from = from;
        e = launch_levels<1>(mid, cnt, to - 1, stream);
        if (e != hipSuccess) return e;
        e = launch_solve(&bands_solve_kernel<PPO_MAX_K, kTail, false>, allowed[2], p, (uint32_t)cnt, kSubsetMaxWaves, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ppo
