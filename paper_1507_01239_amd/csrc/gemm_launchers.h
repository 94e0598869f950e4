// Launch wrappers of the GEMM kernel families.  Each family is instantiated in a translation unit of its own
// (gemm_split*.hip, gemm_dma64.hip, gemm_kg.hip, gemm_kg64.hip, gemm_legacy.hip); gemm.hip plans and dispatches.
#pragma once
#include "gemm_device.h"

namespace mavg {

// register-staged kernels, 64x64 tiles
void launch_legacy(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_grouped_legacy(const GemmGroupParams& gp, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
// direct-to-LDS kernels: 64x64 tiles with a ring of 4 (CFG_64) or 3 (CFG_64_RING3) stages
void launch_dma64(int cfg, const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_grouped_dma(const GemmGroupParams& gp, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
// contraction split inside the workgroup: 32x64 tiles (CFG_KG_32x64) or 32x32 tiles (CFG_KG_32x32); thin grouped problems
void launch_kg(int cfg, const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
// ... and of 64x64 and 64x128 tiles (CFG_KG_64x64, CFG_KG_64x128)
void launch_kg64(int cfg, const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
// split-operand kernels: two fp16 parts per fp32 element, three bf16 parts, or as the data ask for; grouped: m- and n-contiguous
// operands only, `wide`: 256x128 tiles
void launch_split256(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split128(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split64x128(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split64(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split32x64(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_grouped_split(const GemmGroupParams& gp, bool wide, dim3 grid, hipStream_t s);
void launch_split256_three(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split128_three(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split64x128_three(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split64_three(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split32x64_three(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_grouped_split_three(const GemmGroupParams& gp, bool wide, dim3 grid, hipStream_t s);
void launch_split256_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split128_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split64x128_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split64_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_split32x64_by_data(const GemmKParams& p, bool a_kc, bool b_kc, dim3 grid, hipStream_t s);
void launch_grouped_split_by_data(const GemmGroupParams& gp, bool wide, dim3 grid, hipStream_t s);
void launch_thin(const ThinGroupParams& gp, dim3 grid, hipStream_t s);

}  // namespace mavg
