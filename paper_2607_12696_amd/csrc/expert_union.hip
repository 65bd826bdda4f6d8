// moe_expert_union: the expert union, counts, offsets and stable grouping of the
// routed slots, in one workgroup (union_block.hpp).
#include "launch.hpp"
#include "union_block.hpp"

namespace ecospec {

__global__ __launch_bounds__(kUnionThreads) void expert_union_kernel(
    const int32_t *__restrict__ idx, int S, int E, int32_t *__restrict__ counts, int32_t *__restrict__ union_ids,
    int32_t *__restrict__ n_unique, int32_t *__restrict__ offsets, int32_t *__restrict__ perm)
{
    __shared__ UnionLds L;
    union_block(L, idx, S, E, counts, union_ids, n_unique, offsets, perm);
}

hipError_t launch_expert_union(const int32_t *idx, int T, int k, int E, int32_t *counts, int32_t *union_ids,
                               int32_t *n_unique, int32_t *offsets, int32_t *perm, hipStream_t stream)
{
    hipLaunchKernelGGL(expert_union_kernel, dim3(1), dim3(kUnionThreads), 0, stream, idx, T * k, E, counts,
                       union_ids, n_unique, offsets, perm);
    return hipGetLastError();
}

}  // namespace ecospec
