// Split-operand GEMM kernels (gemm_split.h): 256x128 tiles, two fp16 parts or three bf16 parts.
#include "gemm_split.h"
#include "gemm_launchers.h"

namespace mavg {

void launch_split256_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s) { launch_split<kPartsByData, 256, 128, 4, 2, 1>(p, a_kc, b_kc, grid, s); }

}  // namespace mavg
