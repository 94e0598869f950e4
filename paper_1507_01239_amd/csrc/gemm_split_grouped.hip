// Grouped split-operand GEMM (gemm_split.h): the weight gradients of all layers in one launch.
#include "gemm_split.h"
#include "gemm_launchers.h"

namespace mavg {

void launch_grouped_split(const GemmGroupParams& gp, dim3 grid, hipStream_t s) {
    hipLaunchKernelGGL((gemm_split_grouped_kernel<128, 128, 2, 2, 1, 2, false, false>), grid, dim3(256), 0, s, gp);
}

}  // namespace mavg
