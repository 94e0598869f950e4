// Device side of the weight updates C = beta C + alpha A^T B on the fp16 matrix cores, with both operands split into their two fp16
// parts beforehand, by a launch of its own (pack_kernel in gemm_packed.hip).
//
// Why beforehand: a weight update contracts over the minibatch, so its operands (activations and output errors) are small next to
// its output, and every element of them is used in as many tiles as the other operand has tile columns: 16 to 63 times in the
// 440-6x2048-8000 network.  Split on the way into LDS (gemm_split.h), an element costs its 15 - 20 cycles of vector
// instructions in each of them, and the kernel waits for those, not for the matrix pipe.  Packed operands go from memory straight into LDS
// and from LDS straight into the matrix instructions.
//
// Packed form of a matrix X of `rows` contraction steps and `cols` columns: k-tiles of 16 rows; in each two planes (high, low parts), in each
// two halves of 8 rows, in each for every column the 8 rows' parts next to each other, 16 bytes.  That is the order in which the
// lanes of a 32x32x16 MFMA hold an operand, and 64 columns of one half are one direct load of a wavefront (1 KB), whatever the
// alignment of X.  Rows past the last are zeros.
// Every column is scaled by a power of two of its own, so that its largest magnitude lies in [2^14, 2^15): x 2^e = h + l 2^-11, h = fp16(x 2^e),
// l = fp16((x 2^e - h) 2^11), both rounded to nearest, which is off by at most 2^-23 of x (2^-51 of the column's largest where
// that is more), whatever the column's magnitude.  h h' is accumulated in one set of registers, h l' + l h' in another, l l' is
// left out: the errors of the two-part form in gemm_split.h, for operands of any range.
// An infinity or a NaN leaves one in every accumulator that its column takes part in; such blocks are computed again by fp32 MFMAs from
// the operands as they were.
#pragma once
#include "gemm_device.h"

namespace mavg {

struct PackedParams {
    GemmKParams g;                       // the problem as gemm_split.h has it (A, B: the operands as they were)
    const char* pa; const char* pb;      // packed operands
    int64_t pa_bstride, pb_bstride;      // bytes
    const int32_t* ea; const int32_t* eb;       // the columns' exponents, readable up to a multiple of 256
    int64_t e_bstride_a, e_bstride_b;
    int kt;                              // k-tiles
    const float* A2; const float* B2;    // the operands' second pieces, or null
    int64_t lda2, ldb2;
};
struct PackedGroupParams {
    PackedParams g[kMaxGroups];
    int tile_start[kMaxGroups + 1];
    int ngroups;
};

// One matrix to pack: `rows` contraction steps, or two pieces of as many (src2: the second one; each is filled up to whole k-tiles).
// Optionally the (weighted) sums of its columns s[b][j], of two pieces the first one's plus sum_sign2 times the second one's:
//   sum_dst[b][j] = sum_beta sum_dst[b][j] + sum_alpha alpha_dev0[b] alpha_dev1[b] s[b][j];  sum_dst2[b][j] += sum_dst[b][j]
// and, of two pieces, per workgroup the sum of the squares of what is summed there.
struct PackMatrix {
    const float* src; int64_t ld, bstride;
    const float* src2; int64_t ld2;
    char* dst; int64_t dst_bstride;
    int32_t* exps; int64_t e_bstride;
    int rows, cols, batch;
    float sum_alpha, sum_beta, sum_sign2;
    float* sum_dst; int64_t sum_bstride;
    float* sum_dst2; int64_t sum2_bstride;
    const float* sum_w; int64_t sum_w_bstride;
    const float* alpha_dev0; const float* alpha_dev1;
    float* sq_partial;
};
constexpr int kMaxPack = 2 * kMaxGroups;
struct PackGroupParams {
    PackMatrix g[kMaxPack];
    int block_start[kMaxPack + 1];      // in workgroups
    int ngroups;
};

// width: columns per workgroup (64, 32 or 16); pieces: 1 or 2, of all matrices
void launch_pack(const PackGroupParams& gp, int width, int pieces, int most_rows, dim3 grid, hipStream_t s);
// tile shapes of the products
constexpr struct { int bm, bn; } kPackedTiles[] = {{64, 64}, {64, 128}, {128, 128}};
constexpr int kPackedShapes = (int)(sizeof kPackedTiles / sizeof kPackedTiles[0]);
void launch_grouped_packed(const PackedGroupParams& gp, int shape, dim3 grid, hipStream_t s);

template <int N>
__device__ __forceinline__ void wait_loads() {      // ... until at most N of the wavefront's loads are on their way; its LDS reads are done
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// The update of a tile that lies wholly inside C, in rows of whole cache lines.  Parameters are read once and written once per call, so both go past the L2s, which
// then keep the packed operands: 87 against 62 us for the seven updates of 440-6x2048-8000 with 16 rows (306 MB of parameters
// read and written, 4.9 TB/s; a copy runs at 4.94), 126 against 96 with 256.  (Parts of lines are better left to the L2s:
// 429-3x1021-3003 at 200 rows 23.9 us this way, 19.7 as write_tile does it.)
template <int TM, int TN>
__device__ __forceinline__ void update_inner(const floatx16 (&acc)[TM][TN], const EpiCtx& c, float beta, int64_t ldc, int64_t ldc2, int mb, int nb, int lrow, int lcol) {
    const uint32_t off = (uint32_t)(((int64_t)(4 * lrow) * ldc + nb + lcol) * 4), off2 = (uint32_t)(((int64_t)(4 * lrow) * ldc2 + nb + lcol) * 4);
    auto row = [&](auto tc, auto vc) { constexpr int t = decltype(tc)::value, v = decltype(vc)::value; return (int64_t)(mb + t / TN * 32 + 8 * (v >> 2) + (v & 3)); };
    float old[TM * TN][16];
    static_for<TM * TN>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        static_for<16>([&](auto vc) { old[t][decltype(vc)::value] = __builtin_nontemporal_load(at_off(c.C + row(tc, vc) * ldc + t % TN * 32, off)); });
    });
    static_for<TM * TN>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        float old2[16];      // (block by block: registers)
        if (c.C2) static_for<16>([&](auto vc) { old2[decltype(vc)::value] = __builtin_nontemporal_load(at_off(c.C2 + row(tc, vc) * ldc2 + t % TN * 32, off2)); });
        static_for<16>([&](auto vc) {
            constexpr int v = decltype(vc)::value;
            const float r = c.alpha * acc[t / TN][t % TN][v] + beta * old[t][v];
            __builtin_nontemporal_store(r, at_off(c.C + row(tc, vc) * ldc + t % TN * 32, off));
            if (c.C2) __builtin_nontemporal_store(old2[v] + r, at_off(c.C2 + row(tc, vc) * ldc2 + t % TN * 32, off2));
        });
    });
}

// Tiles of (64 TM) x (64 TN) by 2x2 wavefronts, each of TM x TN blocks of 32x32; a ring of NST LDS stages of one k-tile each.
// Wavefront w loads run w (high / low plane, first / second half) of both operands' k-tile.
// Step t: the products of high parts of tile t; wait for tile t + 1 and meet; send for tile t + NST into the stage of tile t, whose
// operands everybody has in registers; the other two thirds of the products, with the operand reads of tile t + 1 between them.
template <int TM, int TN, int NST>
__device__ __forceinline__ void gemm_packed_body(const PackedParams& q, const int tile, const int b) {
    const GemmKParams& p = q.g;
    constexpr int BM = 64 * TM, BN = 64 * TN, RUN_A = BM * 16, RUN_B = BN * 16, STAGE = 4 * (RUN_A + RUN_B), LOADS = TM + TN;
    static_assert(NST >= 2 && BM + BN <= 256, "a ring; one exponent per thread");
    __shared__ __attribute__((aligned(1024))) char S[NST * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane >> 5, lcol = lane & 31;
    const int wm = (wave >> 1) * (32 * TM), wn = (wave & 1) * (32 * TN);
    int tm_i, tn_i;
    tile_coords(p, tile, tm_i, tn_i);
    const int m0 = tm_i * BM, n0 = tn_i * BN;
    const int kt = __builtin_amdgcn_readfirstlane(q.kt);

    // (Columns past the edge repeat the last one; what they come to is not stored.)
    uint32_t voa[TM], vob[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) voa[i] = (uint32_t)(min(m0 + i * 64 + lane, p.M - 1) * 16 + kDmaBias - i * 1024);
#pragma unroll
    for (int i = 0; i < TN; ++i) vob[i] = (uint32_t)(min(n0 + i * 64 + lane, p.N - 1) * 16 + kDmaBias - i * 1024);
    const char* sa = reinterpret_cast<const char*>(uniform_u64(reinterpret_cast<uint64_t>(q.pa + (int64_t)b * q.pa_bstride + (int64_t)wave * p.M * 16 - kDmaBias)));
    const char* sb = reinterpret_cast<const char*>(uniform_u64(reinterpret_cast<uint64_t>(q.pb + (int64_t)b * q.pb_bstride + (int64_t)wave * p.N * 16 - kDmaBias)));
    const int64_t stepa = (int64_t)uniform_u64((uint64_t)p.M * 64), stepb = (int64_t)uniform_u64((uint64_t)p.N * 64);
    const uint32_t la = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(S + wave * RUN_A));
    const uint32_t lb = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(S + 4 * RUN_A + wave * RUN_B));
    // (the exponents: requested ahead of every direct load, needed after the loop)
    int ex = 0;
    if (tid < BM) ex = q.ea[(int64_t)b * q.e_bstride_a + m0 + tid];
    else if (tid < BM + BN) ex = q.eb[(int64_t)b * q.e_bstride_b + n0 + tid - BM];
    auto issue = [&](int t, int stage) {
        const float* ga = reinterpret_cast<const float*>(sa + t * stepa);
        const float* gb = reinterpret_cast<const float*>(sb + t * stepb);
        const uint32_t saved_m0 = m0_swap(la + stage * STAGE);
        static_for<TM>([&](auto ic) { dma16_m0<decltype(ic)::value * 1024>(voa[decltype(ic)::value], ga); });
        m0_set(lb + stage * STAGE);
        static_for<TN>([&](auto ic) { dma16_m0<decltype(ic)::value * 1024>(vob[decltype(ic)::value], gb); });
        m0_set(saved_m0);
    };

    floatx16 acc[TM][TN], low[TM][TN];
    static_for<TM * TN>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        acc[t / TN][t % TN] = low[t / TN][t % TN] = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    });
    const char* ra = S + lrow * RUN_A + (wm + lcol) * 16;
    const char* rb = S + 4 * RUN_A + lrow * RUN_B + (wn + lcol) * 16;
    halfx8 fa[2][2][TM], fb[2][2][TN];      // [set][plane][block]
    constexpr int READS = 2 * (TM + TN);
    auto read_frag = [&](auto ic, auto setc, auto stagec) {      // high parts first
        constexpr int I = decltype(ic)::value, set = decltype(setc)::value, st = decltype(stagec)::value, pl = I / (TM + TN), r = I % (TM + TN);
        if constexpr (r < TM) fa[set][pl][r] = *reinterpret_cast<const halfx8*>(ra + st * STAGE + pl * 2 * RUN_A + r * 512);
        else fb[set][pl][r - TM] = *reinterpret_cast<const halfx8*>(rb + st * STAGE + pl * 2 * RUN_B + (r - TM) * 512);
    };
#pragma unroll
    for (int t = 0; t < NST; ++t)
        if (t < kt) issue(t, t);
    if (kt >= NST) wait_loads<(NST - 1) * LOADS>();
    else wait_loads<0>();
    __syncthreads();
    static_for<READS>([&](auto ic) { read_frag(ic, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}); });
    auto step = [&](auto uc, const int t) {
        constexpr int u = decltype(uc)::value, set = u & 1, cur = u % NST, nxt = (u + 1) % NST, NMF = 2 * TM * TN;
        static_for<TM * TN>([&](auto qc) {
            constexpr int i = decltype(qc)::value / TN, j = decltype(qc)::value % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[set][0][i], fb[set][0][j], acc[i][j], 0, 0, 0);
        });
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < kt) {
            if (t + NST <= kt) wait_loads<(NST - 2) * LOADS>();      // (tiles up to t + NST - 1 have been sent for)
            else wait_loads<0>();
            __syncthreads();
            if (t + NST < kt) issue(t + NST, cur);
        }
        __builtin_amdgcn_sched_barrier(0);
        static_for<NMF>([&](auto qc) {
            constexpr int qq = decltype(qc)::value, pr = qq / (TM * TN), i = qq / TN % TM, j = qq % TN;
            low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[set][1 - pr][i], fb[set][pr][j], low[i][j], 0, 0, 0);
            constexpr int r0 = qq * READS / NMF, r1 = (qq + 1) * READS / NMF;
            // (behind the last step: what an earlier tile left there, and nobody uses)
            static_for<r1 - r0>([&](auto ic) { read_frag(std::integral_constant<int, r0 + decltype(ic)::value>{}, std::integral_constant<int, set ^ 1>{}, std::integral_constant<int, nxt>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    constexpr int PERIOD = NST % 2 ? 2 * NST : NST;
    for (int t = 0; t < kt; t += PERIOD)
        static_for<PERIOD>([&](auto uc) { if (t + decltype(uc)::value < kt) step(uc, t + decltype(uc)::value); });

    __syncthreads();
    int* es = reinterpret_cast<int*>(S);
    if (tid < BM + BN) es[tid] = ex;
    __syncthreads();
    static_for<TM * TN>([&](auto tc) {
        constexpr int i = decltype(tc)::value / TN, j = decltype(tc)::value % TN;
        static_for<16>([&](auto vc) { constexpr int v = decltype(vc)::value; acc[i][j][v] = __builtin_fmaf(low[i][j][v], 0x1p-11f, acc[i][j][v]); });
        if (block_suspect(acc[i][j])) {
            const float *Ab = p.A + (int64_t)b * p.a_bstride, *Bb = p.B + (int64_t)b * p.b_bstride;
            acc[i][j] = block_fp32<false, false>(Ab, p.lda, Bb, p.ldb, p.M, p.N, m0 + wm + 32 * i, n0 + wn + 32 * j, 0, p.K, 1);
            if (q.A2) acc[i][j] += block_fp32<false, false>(q.A2, q.lda2, q.B2, q.ldb2, p.M, p.N, m0 + wm + 32 * i, n0 + wn + 32 * j, 0, p.K, 1);
        } else {
            const int eb = es[BM + wn + 32 * j + lcol];
            static_for<16>([&](auto vc) {
                constexpr int v = decltype(vc)::value;
                acc[i][j][v] = __builtin_ldexpf(acc[i][j][v], -(es[wm + 32 * i + 8 * (v >> 2) + 4 * lrow + (v & 3)] + eb));
            });
        }
    });
    const EpiCtx c = epi_ctx(p.epi, p.C, p.c_bstride, b);
    const auto whole_lines = [](const float* q, int64_t ld) { return ((reinterpret_cast<uint64_t>(q) | (uint64_t)ld * 4) & 127) == 0; };
    if (p.epi.beta != 0.f && m0 + BM <= p.M && n0 + BN <= p.N && whole_lines(c.C, p.ldc) && (!c.C2 || whole_lines(c.C2, p.epi.ldc2)))
        update_inner<TM, TN>(acc, c, p.epi.beta, p.ldc, p.epi.ldc2, m0 + wm, n0 + wn, lrow, lcol);
    else
        write_tile<EPI_AXPBY, TM, TN>(acc, p.epi, c, p.ldc, p.M, p.N, m0 + wm, n0 + wn, lrow, lcol);
    if (p.epi.side_sum_src != nullptr && tile == 0 && b == 0) side_sum(p.epi, reinterpret_cast<float*>(S));      // (uniform over the workgroup)
}

}  // namespace mavg
