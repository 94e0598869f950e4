// Split-operand GEMM kernels (gemm_split.h): 32x64 tiles, two fp16 parts or three bf16 parts.
#include "gemm_split.h"
#include "gemm_launchers.h"

namespace mavg {

void launch_split32x64_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s) { launch_split<kPartsByData, 32, 64, 1, 1, 8>(p, a_kc, b_kc, grid, s); }

}  // namespace mavg
