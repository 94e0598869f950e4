// Split-operand GEMM kernels (gemm_split.h): 128x128 tiles, two k-groups.
#include "gemm_split.h"
#include "gemm_launchers.h"

namespace mavg {

void launch_split128(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s) {
    const dim3 block(512);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_split_kernel<128, 128, 2, 2, 2, 2, true, true>), grid, block, 0, s, p);
    else if (a_kc && !b_kc) hipLaunchKernelGGL((gemm_split_kernel<128, 128, 2, 2, 2, 2, true, false>), grid, block, 0, s, p);
    else if (!a_kc && !b_kc) hipLaunchKernelGGL((gemm_split_kernel<128, 128, 2, 2, 2, 2, false, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_split_kernel<128, 128, 2, 2, 2, 2, false, true>), grid, block, 0, s, p);
}

}  // namespace mavg
