// Host interface of the weight updates on packed operands (gemm_packed.h).
#pragma once
#include "gemm.h"

namespace mavg {

// The operands' second pieces, where a contraction runs over two of K steps each, and what else the launch that packs leaves: of the
// differences of B's pieces the column sums, diff_dst = diff_beta diff_dst + diff_alpha sum, diff_dst2 += diff_dst, and the sum of
// squares.  (Epilogue::rowsum_* are the sums over both pieces of A.)
struct PackedPieces {
    const float* A2 = nullptr; int64_t lda2 = 0;
    const float* B2 = nullptr; int64_t ldb2 = 0;
    float* diff_dst = nullptr; float diff_alpha = 1.f, diff_beta = 0.f; float* diff_dst2 = nullptr;
    float* square_dst = nullptr;      // (null: not wanted)
};

// C[b] = beta C[b] + alpha A[b]^T B[b] for several problems with m- and n-contiguous operands (EPI_AXPBY) and the same batch count: one launch
// that packs the operands into two fp16 parts, one for the products.  Needs the sum of gemm_packed_floats() of scratch,
// 16-byte aligned.  gemm_packed_takes: is that the faster way, and no less exact?  tiles: which tile shape (-1: choose).
int64_t gemm_packed_floats(int M, int N, int K, int batch, int pieces = 1);
bool gemm_packed_takes(const GemmDesc* d, int count, int pieces = 1);
int gemm_launch_packed(const GemmDesc* d, int count, float* ws, int64_t ws_floats, hipStream_t stream, int tiles = -1, const PackedPieces* pieces = nullptr);

}  // namespace mavg
