// Kernels of single fp32 problems on the bf16 matrix units.
#include "gemm_split.hpp"

namespace adpsgd {
namespace {

template <bool AKC, bool BKC, int F>
__global__ __launch_bounds__(256, 3) void gemm_split_kernel(GemmDesc p) {
    __shared__ __attribute__((aligned(1024))) char lds[SplitCore<AKC, BKC, F>::LDS_BYTES];
    split_tile<AKC, BKC, F>(p, blockIdx.x, gridDim.x, lds);
}

template <int F> hipError_t launch_f(const GemmDesc& d, hipStream_t s) {
    const int64_t tiles = (int64_t)((d.M + 64 * F - 1) / (64 * F)) * ((d.N + 64 * F - 1) / (64 * F)) * d.groupsI * d.groupsD;
    const dim3 grid((unsigned)tiles);
    switch ((d.a_kc ? 2 : 0) | (d.b_kc ? 1 : 0)) {
        case 0: hipLaunchKernelGGL((gemm_split_kernel<false, false, F>), grid, dim3(256), 0, s, d); break;
        case 1: hipLaunchKernelGGL((gemm_split_kernel<false, true, F>), grid, dim3(256), 0, s, d); break;
        case 2: hipLaunchKernelGGL((gemm_split_kernel<true, false, F>), grid, dim3(256), 0, s, d); break;
        default: hipLaunchKernelGGL((gemm_split_kernel<true, true, F>), grid, dim3(256), 0, s, d); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_split(const GemmDesc& d, bool large, hipStream_t s) { return large ? launch_f<2>(d, s) : launch_f<1>(d, s); }

}  // namespace adpsgd
