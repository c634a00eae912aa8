// The paper's partitioning step on its own (Sec. III-B1, Alg. 1): cut the chain into segments that each fit a
// node of capacity kappa so that the SUM of the transfer sizes at the cuts is least (the path of least cost
// through the partition graph, whose vertices are the contiguous runs of partition points that fit and whose
// edge weights are the transfer sizes).  With f[i] = least sum for layers [i, L):
//     f[L] = 0,   f[i] = min over e in (i, L] with layers [i, e) fitting   of   (e < L ? t[e-1] : 0) + f[e].
// One wave per instance (ppo_partition.h); sums in binary64, added from the chain's end.
#include "ppo_partition.h"

namespace ppo {

__global__ __launch_bounds__(64) void min_sum_partition_kernel(const float* __restrict__ t, const float* __restrict__ m,
                                                               int L, const float* __restrict__ kappa,
                                                               int32_t* __restrict__ segs_out,
                                                               int32_t* __restrict__ cuts_out,
                                                               double* __restrict__ sum_out) {
    __shared__ PartitionShared S;
    const int inst = blockIdx.x, lane = threadIdx.x;
    double sum;
    const int segs = min_sum_partition_wave(t + (size_t)inst * L, m + (size_t)inst * L, L, (double)kappa[inst], lane, S, sum);
    int32_t* cuts = cuts_out + (size_t)inst * (L - 1);
    for (int i = lane; i < L - 1; i += 64) cuts[i] = i + 1 < segs ? (int32_t)S.cut[i] : -1;
    if (lane == 0) {
        sum_out[inst] = sum;
        segs_out[inst] = segs;
    }
}

hipError_t launch_min_sum_partition(const float* t, const float* m, int L, const float* kappa, int n_inst,
                                    int32_t* segs_out, int32_t* cuts_out, double* sum_out, hipStream_t stream) {
    hipLaunchKernelGGL(min_sum_partition_kernel, dim3(n_inst), dim3(64), 0, stream, t, m, L, kappa, segs_out, cuts_out,
                       sum_out);
    return hipGetLastError();
}

}  // namespace ppo
