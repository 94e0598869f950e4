// Split-operand GEMM kernels (gemm_split.h): several problems in one launch, 128x128 or 256x128 tiles, two fp16 parts or three bf16 parts.
#include "gemm_split.h"
#include "gemm_launchers.h"

namespace mavg {

void launch_grouped_split_by_data(const GemmGroupParams& gp, bool wide, dim3 grid, hipStream_t s) {
    if (wide) hipLaunchKernelGGL((gemm_split_grouped_kernel<kPartsByData, 256, 128, 4, 2, 1, 2, false, false>), grid, dim3(512), 0, s, gp);
    else hipLaunchKernelGGL((gemm_split_grouped_kernel<kPartsByData, 128, 128, 2, 2, 1, 2, false, false>), grid, dim3(256), 0, s, gp);
}

}  // namespace mavg
