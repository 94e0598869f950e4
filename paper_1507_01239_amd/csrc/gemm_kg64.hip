// 64x64 tiles with the contraction split four ways inside the workgroup.
#include "gemm_kg64.h"
#include "gemm_launchers.h"

namespace mavg {

template <bool AKC, bool BKC>
__global__ __launch_bounds__(64 * kKg64Groups, 1) void gemm_kg64_kernel(GemmKParams p) {
    gemm_kg64_body<AKC, BKC>(p, blockIdx.x, blockIdx.z);
}

void launch_kg64(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s) {
    const dim3 block(64 * kKg64Groups);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_kg64_kernel<true, true>), grid, block, 0, s, p);
    else if (a_kc && !b_kc) hipLaunchKernelGGL((gemm_kg64_kernel<true, false>), grid, block, 0, s, p);
    else if (!a_kc && !b_kc) hipLaunchKernelGGL((gemm_kg64_kernel<false, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_kg64_kernel<false, true>), grid, block, 0, s, p);
}

}  // namespace mavg
