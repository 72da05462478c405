// D of the short rows for the rowsum stage (see sp_edge.hpp; their dQ is written by the dq pass's launch).
#include "sp_edge.hpp"

namespace sp {
namespace {

__global__ __launch_bounds__(128) void short_rows_kernel(EdgeArgs a) {
    __shared__ __attribute__((aligned(1024))) char lds[EDGE_LDS];
    for (int64_t pair = blockIdx.x; pair < a.n_pairs; pair += gridDim.x) {
        short_rows_body<false>(a, pair, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lds);
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_short_rows(const Problem& p, hipStream_t s) {
    const EdgeArgs a = edge_args(p);
    if (a.n_pairs > 0) hipLaunchKernelGGL(short_rows_kernel, dim3(edge_blocks(a, 1)), dim3(128), 0, s, a);
    return hipGetLastError();
}

}  // namespace sp
