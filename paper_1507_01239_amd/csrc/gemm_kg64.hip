// 64x64 tiles with the contraction split four ways inside the workgroup.
#include "gemm_kg64.h"
#include "gemm_launchers.h"

namespace mavg {

template <bool AKC, bool BKC, int TN>
__global__ __launch_bounds__(64 * kKg64Groups, 1) void gemm_kg64_kernel(GemmKParams p) {
    gemm_kg64_body<AKC, BKC, TN>(p, blockIdx.x, blockIdx.z);
}

template <int TN>
static void launch_kg64_t(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s) {
    const dim3 block(64 * kKg64Groups);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_kg64_kernel<true, true, TN>), grid, block, 0, s, p);
    else if (a_kc && !b_kc) hipLaunchKernelGGL((gemm_kg64_kernel<true, false, TN>), grid, block, 0, s, p);
    else if (!a_kc && !b_kc) hipLaunchKernelGGL((gemm_kg64_kernel<false, false, TN>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_kg64_kernel<false, true, TN>), grid, block, 0, s, p);
}

void launch_kg64(int cfg, const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s) {
    if (cfg == CFG_KG_64x64) launch_kg64_t<2>(p, a_kc, b_kc, grid, s);
    else launch_kg64_t<4>(p, a_kc, b_kc, grid, s);
}

}  // namespace mavg
