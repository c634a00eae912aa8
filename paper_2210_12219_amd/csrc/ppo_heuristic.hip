// The two systems that the paper compares its placement algorithm with (Sec. IV): the random and the greedy
// joint-optimisation system.  (The algorithm itself: ppo_kpath.hip.)
//
// One wave per instance; the choices are sequential by nature and run on lane 0.  Not a tuned path.
#include "ppo_common.h"

namespace ppo {

struct HeurShared {
    int node[PPO_MAX_L + 1];            // node of every segment
};

__device__ inline float heur_gamma(float tv, float bw) {
    const float q = __fdiv_rn(tv, bw);
    return q == 0.0f ? 0.0f : q;
}

// mode 1: joint-optimisation system; 2: random system (draws given)
__global__ __launch_bounds__(64) void heuristic_kernel(const float* __restrict__ t, const float* __restrict__ m, int L,
                                                       const float* __restrict__ kappa, const float* __restrict__ Ball,
                                                       int n, int mode, const float* __restrict__ draws, int n_draws,
                                                       float* __restrict__ beta_out, int32_t* __restrict__ segs_out,
                                                       int32_t* __restrict__ cuts_out, int32_t* __restrict__ order_out) {
    __shared__ HeurShared S;
    __shared__ double P[PPO_MAX_L + 1];
    __shared__ int cut_s[PPO_MAX_L];
    __shared__ int p_s;
    const int inst = blockIdx.x, lane = threadIdx.x;
    const float* ti = t + (size_t)inst * L;
    const float* B = Ball + (size_t)inst * n * n;
    int32_t* cuts_o = cuts_out + (size_t)inst * (L > 1 ? L - 1 : 0);
    int32_t* order_o = order_out + (size_t)inst * n;
    const float inf = __uint_as_float(kInfBits);
    for (int i = lane; i < L - 1; i += 64) cuts_o[i] = -1;
    for (int i = lane; i < n; i += 64) order_o[i] = -1;
    __syncthreads();
    auto fail = [&]() {
        if (lane == 0) {
            beta_out[inst] = inf;
            segs_out[inst] = 0;
        }
    };
    // ---- the cuts
    if (lane == 0) {
        const float* mi = m + (size_t)inst * L;
        const double cap = (double)kappa[inst];
        double acc = 0.0;
        P[0] = 0.0;
        for (int i = 0; i < L; ++i) {
            acc = acc + (double)mi[i];
            P[i + 1] = acc;
        }
        int p = 0, i = 0, d = 0;
        unsigned long long free_nodes = n < 64 ? (1ull << n) - 1ull : ~0ull;
        bool ok = true;
        while (i < L && ok) {
            int last = i;   // the last end that fits
            while (last < L && (P[last + 1] - P[i]) <= cap) ++last;
            if (last == i) { ok = false; break; }
            int e;
            if (mode == 1) {
                // the fitting end with the smallest transfer size; the rest of the chain as soon as it fits
                e = last;
                if (last < L) {
                    e = i + 1;
                    for (int x = i + 2; x <= last; ++x)
                        if (ti[x - 1] < ti[e - 1]) e = x;
                }
            } else {
                // a random free node, then a random fitting end
                const int nfree = __popcll(free_nodes);
                if (nfree == 0 || d + 1 >= n_draws) { ok = false; break; }
                int pick = (int)((double)draws[(size_t)inst * n_draws + d] * (double)nfree);
                unsigned long long f = free_nodes;
                for (int s = 0; s < pick; ++s) f &= f - 1ull;
                const int node = __ffsll((long long)f) - 1;
                free_nodes &= ~(1ull << node);
                S.node[p] = node;
                e = i + 1 + (int)((double)draws[(size_t)inst * n_draws + d + 1] * (double)(last - i));
                d += 2;
            }
            if (e < L) cut_s[p] = e;
            ++p;
            i = e;
        }
        p_s = ok ? p : 0;
    }
    __syncthreads();
    const int p = p_s;
    if (p == 0 || p > n) { fail(); return; }
    if (mode == 1) {
        // ---- joint system: from every start node, always on over the best link to a free node; the best start
        if (lane == 0) {
            float best_beta = inf;
            int best_first = 0;   // also if a quotient of every start overflows to +inf
            for (int first = 0; first < n; ++first) {
                unsigned long long used = 1ull << first;
                int cur = first;
                float beta = 0.0f;
                for (int s = 1; s < p; ++s) {
                    int nxt = -1;
                    for (int v = 0; v < n; ++v)
                        if (!((used >> v) & 1ull) && (nxt < 0 || B[cur * n + v] > B[cur * n + nxt])) nxt = v;
                    const float g = heur_gamma(ti[cut_s[s - 1] - 1], B[cur * n + nxt]);
                    beta = g > beta ? g : beta;
                    used |= 1ull << nxt;
                    cur = nxt;
                }
                if (beta < best_beta) { best_beta = beta; best_first = first; }
            }
            unsigned long long used = 1ull << best_first;
            S.node[0] = best_first;
            for (int s = 1; s < p; ++s) {
                const int cur = S.node[s - 1];
                int nxt = -1;
                for (int v = 0; v < n; ++v)
                    if (!((used >> v) & 1ull) && (nxt < 0 || B[cur * n + v] > B[cur * n + nxt])) nxt = v;
                S.node[s] = nxt;
                used |= 1ull << nxt;
            }
        }
    }
    __syncthreads();
    // ---- Eq. 2, Eq. 3 of the placement found
    if (lane == 0) {
        float beta = 0.0f;
        for (int s = 1; s < p; ++s) {
            const float g = heur_gamma(ti[cut_s[s - 1] - 1], B[S.node[s - 1] * n + S.node[s]]);
            beta = g > beta ? g : beta;
        }
        beta_out[inst] = beta;
        segs_out[inst] = p;
        for (int s = 0; s < p; ++s) order_o[s] = S.node[s];
        for (int s = 0; s + 1 < p; ++s) cuts_o[s] = cut_s[s];
    }
}

hipError_t launch_heuristic(const float* t, const float* m, int L, const float* kappa, const float* B, int n, int n_inst,
                            int mode, const float* draws, int n_draws, float* beta_out, int32_t* segs_out, int32_t* cuts_out,
                            int32_t* order_out, hipStream_t stream) {
    hipLaunchKernelGGL(heuristic_kernel, dim3(n_inst), dim3(64), 0, stream, t, m, L, kappa, B, n, mode, draws, n_draws,
                       beta_out, segs_out, cuts_out, order_out);
    return hipGetLastError();
}

}  // namespace ppo
