// Weight updates on packed operands (gemm_packed.h): the launch that packs them, and the grouped products.
#include "gemm_packed.h"
#include "gemm_launchers.h"

namespace mavg {

// ---- packing ---------------------------------------------------------------------------------------
// A workgroup of 512 threads packs C columns, 512 / C groups of eight rows of each at a time; a thread keeps the G groups that it gets in
// registers (0: any number; the columns are then read twice).  The columns' largest magnitudes
// and sums meet in LDS.  64 columns read whole cache lines, 440-6x2048-8000 with 1000 rows 264 MB in 54 us; 16 columns give few of them
// enough workgroups: 440 + 2048 columns of 1000 rows 15 us with 64.
template <int C, int G, int SEG>
__global__ __launch_bounds__(512) void pack_kernel(PackGroupParams gp) {
    constexpr int RG = 512 / C;
    __shared__ float tops[8][C];
    __shared__ float sums[8][C], sq[8];
    int gi = 0, first = 0;
    static_for<kMaxPack - 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value + 1;
        if (i < gp.ngroups && (int)blockIdx.x >= gp.block_start[i]) { gi = i; first = gp.block_start[i]; }
    });
    gi = __builtin_amdgcn_readfirstlane(gi);
    typedef const __attribute__((address_space(4))) char* ConstBytes;      // (the record in the kernel-argument segment, see group_params)
    typedef const __attribute__((address_space(4))) PackMatrix* ConstMatrix;
    const PackMatrix& m = *(const PackMatrix*)(ConstMatrix)((ConstBytes)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PackGroupParams, g) +
                                                           (size_t)gi * sizeof(PackMatrix));
    const int b = blockIdx.y, block = (int)blockIdx.x - first;
    if (b >= m.batch) return;      // (uniform: an operand that all replicas share is packed once)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = tid % C, rg = C == 64 ? wave : tid / C;
    const int col = block * C + c, cols = m.cols, rows = m.rows;
    const bool col_ok = col < cols;
    const int colr = min(col, cols - 1);
    const int groups = (rows + 15) / 16 * 2;      // of eight rows, per piece
    const float* w = m.sum_w ? m.sum_w + (int64_t)b * m.sum_w_bstride : nullptr;

    auto load = [&](int seg, int g, float (&x)[8]) {
        const int64_t ld = (int64_t)uniform_u64((uint64_t)(seg ? m.ld2 : m.ld));
        const float* r = (seg ? m.src2 : m.src + (int64_t)b * m.bstride) + (int64_t)g * 8 * ld;
        if (g * 8 + 8 <= rows) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = (r + (int64_t)j * ld)[(uint32_t)colr];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = g * 8 + j < rows ? (r + (int64_t)j * ld)[(uint32_t)colr] : 0.f;
        }
    };
    float top = 0.f;      // (NaNs are passed over: they are NaNs at any scale)
    float sum = 0.f, squares = 0.f;
    auto look = [&](int seg, int g, const float (&x)[8]) {
#pragma unroll
        for (int j = 0; j < 8; j += 2) most_of(top, x[j], x[j + 1]);
        if (m.sum_dst && SEG == 1) {
            if (w) {
#pragma unroll
                for (int j = 0; j < 8; ++j) if (g * 8 + j < rows) sum += x[j] * w[g * 8 + j];
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) sum += x[j];
            }
        }
    };
    auto combine = [&](const float (&x)[8], const float (&y)[8]) {      // (a thread has the same rows of both pieces)
#pragma unroll
        for (int j = 0; j < 8; ++j) { const float d = x[j] + m.sum_sign2 * y[j]; sum += d; squares += d * d; }
    };
    float x[SEG][G > 0 ? G : 1][8];
    if constexpr (G > 0) {
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int s = 0; s < SEG; ++s)
                if (rg + RG * i < groups) load(s, rg + RG * i, x[s][i]);
#pragma unroll
        for (int i = 0; i < G; ++i)
            if (rg + RG * i < groups) {
#pragma unroll
                for (int s = 0; s < SEG; ++s) look(s, rg + RG * i, x[s][i]);
                if constexpr (SEG == 2) if (m.sum_dst) combine(x[0][i], x[1][i]);
            }
    } else {
        for (int g = rg; g < groups; g += RG) {
#pragma unroll
            for (int s = 0; s < SEG; ++s) { load(s, g, x[s][0]); look(s, g, x[s][0]); }
            if constexpr (SEG == 2) if (m.sum_dst) combine(x[0][0], x[1][0]);
        }
    }
#pragma unroll
    for (int o = C; o < 64; o *= 2) top = fmaxf(top, __shfl_xor(top, o, 64));
    if (lane < C) tops[wave][c] = top;
    if (m.sum_dst) {
#pragma unroll
        for (int o = C; o < 64; o *= 2) sum += __shfl_xor(sum, o, 64);
        if (lane < C) sums[wave][c] = sum;
        if (SEG == 2 && m.sq_partial) {
            const float s = wave_sum(col_ok ? squares : 0.f);
            if (lane == 0) sq[wave] = s;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) top = fmaxf(top, tops[i][c]);
    // the exponent that brings the largest magnitude into [2^14, 2^15); none for zeros and infinities
    const int e = top > 0.f && top < INFINITY ? 15 - __builtin_amdgcn_frexp_expf(top) : 0;
    if (tid < C && col_ok) {
        m.exps[(int64_t)b * m.e_bstride + col] = e;
        if (m.sum_dst) {
            float s = sums[0][c];
#pragma unroll
            for (int i = 1; i < 8; ++i) s += sums[i][c];
            float r = m.sum_alpha * s;
            if (m.alpha_dev0) r *= m.alpha_dev0[b];
            if (m.alpha_dev1) r *= m.alpha_dev1[b];
            float* d = m.sum_dst + (int64_t)b * m.sum_bstride + col;
            if (m.sum_beta != 0.f) r += m.sum_beta * *d;
            *d = r;
            if (m.sum_dst2) m.sum_dst2[(int64_t)b * m.sum2_bstride + col] += r;
        }
    }
    if (SEG == 2 && m.sq_partial && tid == 0) m.sq_partial[block] = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
    char* const dst = m.dst + (int64_t)b * m.dst_bstride + (int64_t)col * 16;
    auto store = [&](int seg, int g, float (&v)[8]) {
        uint32_t h[4], l[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float x0 = __builtin_ldexpf(v[2 * j], e), x1 = __builtin_ldexpf(v[2 * j + 1], e);
            split_step<0, false>(x0, x1, h[j], l[j], 1.f);
            split_step<1, false>(x0, x1, h[j], l[j], 1.f);
            split_step<2, false>(x0, x1, h[j], l[j], 1.f);
        }
        const int at = seg * groups + g;
        char* const d = dst + ((int64_t)(at >> 1) * 4 + (at & 1)) * cols * 16;
        if (col_ok) {
            *reinterpret_cast<uintx4*>(d) = uintx4{h[0], h[1], h[2], h[3]};
            *reinterpret_cast<uintx4*>(d + (int64_t)cols * 32) = uintx4{l[0], l[1], l[2], l[3]};
        }
    };
    if constexpr (G > 0) {
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int s = 0; s < SEG; ++s)
                if (rg + RG * i < groups) store(s, rg + RG * i, x[s][i]);
    } else {
        for (int g = rg; g < groups; g += RG)
#pragma unroll
            for (int s = 0; s < SEG; ++s) { load(s, g, x[s][0]); store(s, g, x[s][0]); }
    }
}

template <int C, int SEG>
static void launch_pack_width(const PackGroupParams& gp, int most_rows, dim3 grid, hipStream_t s) {
    const int groups = (most_rows + 15) / 16 * 2, each = (groups + 512 / C - 1) / (512 / C);
    if (each <= 1) hipLaunchKernelGGL((pack_kernel<C, 1, SEG>), grid, dim3(512), 0, s, gp);
    else if (each <= 2) hipLaunchKernelGGL((pack_kernel<C, 2, SEG>), grid, dim3(512), 0, s, gp);
    else if (each <= 4) hipLaunchKernelGGL((pack_kernel<C, 4, SEG>), grid, dim3(512), 0, s, gp);
    else if (each <= 8) hipLaunchKernelGGL((pack_kernel<C, 8, SEG>), grid, dim3(512), 0, s, gp);
    else if (SEG == 1 && each <= 16) hipLaunchKernelGGL((pack_kernel<C, SEG == 1 ? 16 : 8, SEG>), grid, dim3(512), 0, s, gp);
    else hipLaunchKernelGGL((pack_kernel<C, 0, SEG>), grid, dim3(512), 0, s, gp);
}

void launch_pack(const PackGroupParams& gp, int width, int pieces, int most_rows, dim3 grid, hipStream_t s) {
    if (pieces == 2) (width == 64 ? launch_pack_width<64, 2> : width == 32 ? launch_pack_width<32, 2> : launch_pack_width<16, 2>)(gp, most_rows, grid, s);
    else (width == 64 ? launch_pack_width<64, 1> : width == 32 ? launch_pack_width<32, 1> : launch_pack_width<16, 1>)(gp, most_rows, grid, s);
}

// ---- products --------------------------------------------------------------------------------------
template <int TM, int TN, int NST, int OCC>
__global__ __launch_bounds__(256, OCC) void gemm_packed_grouped_kernel(PackedGroupParams gp) {
    int gi = 0, first = 0;
    static_for<kMaxGroups - 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value + 1;
        if (i < gp.ngroups && (int)blockIdx.x >= gp.tile_start[i]) { gi = i; first = gp.tile_start[i]; }
    });
    gi = __builtin_amdgcn_readfirstlane(gi);
    typedef const __attribute__((address_space(4))) char* ConstBytes;
    typedef const __attribute__((address_space(4))) PackedParams* ConstParams;
    const PackedParams& q = *(const PackedParams*)(ConstParams)((ConstBytes)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PackedGroupParams, g) +
                                                               (size_t)gi * sizeof(PackedParams));
    gemm_packed_body<TM, TN, NST>(q, (int)blockIdx.x - first, blockIdx.z);
}

void launch_grouped_packed(const PackedGroupParams& gp, int shape, dim3 grid, hipStream_t s) {
    if (shape == 0) hipLaunchKernelGGL((gemm_packed_grouped_kernel<1, 1, 4, 4>), grid, dim3(256), 0, s, gp);
    else if (shape == 1) hipLaunchKernelGGL((gemm_packed_grouped_kernel<1, 2, 4, 3>), grid, dim3(256), 0, s, gp);
    else hipLaunchKernelGGL((gemm_packed_grouped_kernel<2, 2, 5, 2>), grid, dim3(256), 0, s, gp);
}

}  // namespace mavg
