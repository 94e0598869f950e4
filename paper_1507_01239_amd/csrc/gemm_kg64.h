// 64x64 and 64x128 tiles, the contraction split four ways inside the workgroup: one wavefront per k-group and SIMD (see gemm_dma_kg_body, of
// which these are the forms for two and four times as many tiles).
#pragma once
#include "gemm_device.h"

namespace mavg {

constexpr int kKg64Groups = 4;

template <int N>
__device__ __forceinline__ void wait_kg64() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// What bounds it: the direct loads, 512 bytes per contraction step and compute unit at 25 bytes a cycle; the loop's 164 instructions per
// k-tile take about half of that time.  512 x 2048 x 2048, k-contiguous / n-contiguous B: 24 / 25 us with B in the last-level cache and 30 / 29
// from HBM, where 128x128 tiles in four splits and their reducer take 33 / 33 and 34 / 34.  (Four stages 25 / 26; the reads at the third or the
// last MFMA instead of behind the eighth 24 / 25; asking for all of B ahead of the loop, and another order of the contraction for every XCD: no gain
// from HBM, the former 25 / 26 otherwise.)
// 64x128 tiles (768 bytes per step for twice the output; 256 accumulation registers, so one set of sums): 1024 x 2048 x 2048 42 / 39 us, from HBM
// 43 / 39, where the split-operand kernel's 64x128 tiles take 48 / 48 and 50 / 50.
// The contraction may be split across workgroups too (fewer tiles, long contractions): 256 x 2048 x 8000, four ways, 42 us and the reducer's 6.6, 128x128 tiles
// in eight splits 48 and 7.6.
// A wavefront's two 32-row blocks of A and two of B make
// four products of every part, so that an element is split half as often per product as in 32x32 blocks side by side, and a compute unit
// reads a third less for the same output than with 32x64 tiles.  A wavefront has its SIMD and 512 registers to itself: k-tile t's
// twelve MFMAs run with the split of tile t + 1 between them, whose raw operands tile t + 2's replace as they are used up.
template <bool AKC, bool BKC, int TN>
__device__ __forceinline__ void gemm_kg64_body(const GemmKParams& p, const int tile, const int bz) {
    // 2 blocks of 32 rows of A, TN blocks of 32 columns of B; sums of even and odd k-tiles apart where there are registers for it (they round less)
    constexpr int KG = kKg64Groups, NST = TN == 2 ? 5 : 3, BK = kDmaBK, BM = 64, BN = 32 * TN, TILE_A = BM * BK, TILE_B = BN * BK;
    constexpr int A_LOADS = 4, B_LOADS = 2 * TN, LOADS = A_LOADS + B_LOADS, BLOCKS = 2 + TN, PRODUCTS = 2 * TN, SETS = TN == 2 ? 2 : 1;
    static_assert(BK == 16 && (TN == 2 || TN == 4), "two pairs of 16-byte chunks per k-tile");
    __shared__ __attribute__((aligned(1024))) float S[KG][NST * (TILE_A + TILE_B)];
    static_assert(NST * (TILE_A + TILE_B) >= PRODUCTS * 1024, "a k-group's rings must hold its accumulators for the final sum");
    const int tid = threadIdx.x, lane = tid & 63, kg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane >> 5, lcol = lane & 31;
    const int b = bz / p.splits, split = bz - b * p.splits;
    int tm_i, tn_i;
    tile_coords(p, tile, tm_i, tn_i);
    const int m0 = tm_i * BM, n0 = tn_i * BN;
    // every KG-th k-tile: what the groups read at a time are neighbouring pieces of the same cache lines
    const int kfirst = split * p.kper, kend = min(p.K, kfirst + p.kper), nkt_all = (kend - kfirst) / BK, ktail = kfirst + nkt_all * BK;
    const int nkt = __builtin_amdgcn_readfirstlane((nkt_all - kg + KG - 1) / KG);
    const int kbeg = kfirst + kg * BK;

    auto lane_offset = [&](bool kc, int unit, int BR, int r0, int R, int64_t ld) -> uint32_t {      // (as in gemm_dma_kg_body)
        if (kc) {
            const int r = unit * 16 + lane / 4, q = (lane % 4) ^ kc_swizzle(r);
            return (uint32_t)(((int64_t)min(r0 + r, R - 1) * ld + q * 4) * 4);
        }
        const int per = BR / 4, k = unit * (256 / BR) + lane / per, col = min(r0 + (lane % per) * 4, R - 4);
        return (uint32_t)(((int64_t)k * ld + col) * 4);
    };
    uint32_t voa[A_LOADS], vob[B_LOADS];
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) voa[i] = lane_offset(AKC, i, BM, m0, AKC ? p.M : p.Mr, p.lda) + kDmaBias - i * 1024;
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) vob[i] = lane_offset(BKC, i, BN, n0, BKC ? p.N : p.Nr, p.ldb) + kDmaBias - i % 4 * 1024;
    const float* sa = reinterpret_cast<const float*>(uniform_u64(reinterpret_cast<uint64_t>(
        p.A + (int64_t)b * p.a_bstride + (AKC ? (int64_t)kbeg : (int64_t)kbeg * p.lda) - kDmaBias / 4)));
    const float* sb = reinterpret_cast<const float*>(uniform_u64(reinterpret_cast<uint64_t>(
        p.B + (int64_t)b * p.b_bstride + (BKC ? (int64_t)kbeg : (int64_t)kbeg * p.ldb) - kDmaBias / 4)));
    const int64_t stepa = (int64_t)uniform_u64((uint64_t)(AKC ? KG * BK : KG * BK * p.lda));
    const int64_t stepb = (int64_t)uniform_u64((uint64_t)(BKC ? KG * BK : KG * BK * p.ldb));
    const uint32_t la = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&S[kg][0]);
    const uint32_t lb = la + NST * TILE_A * 4;
    auto issue = [&](int t, int stage) {
        const float* ga = sa + t * stepa;
        const float* gb = sb + t * stepb;
        const uint32_t saved_m0 = m0_swap(la + stage * (TILE_A * 4));
        static_for<A_LOADS>([&](auto ic) { dma16_m0<decltype(ic)::value * 1024>(voa[decltype(ic)::value], ga); });
        static_for<B_LOADS / 4>([&](auto jc) {      // (immediate offsets of less than 4096)
            constexpr int j = decltype(jc)::value;
            m0_set(lb + stage * (TILE_B * 4) + j * 4096);
            static_for<4>([&](auto ic) { dma16_m0<decltype(ic)::value * 1024>(vob[4 * j + decltype(ic)::value], gb); });
        });
        m0_set(saved_m0);
    };

    // blocks 0, 1: rows of A, from 2 on: columns of B; a lane's eight values are k = 8 pr + 4 lrow + c
    int offa[2], offb[2];
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        offa[pr] = AKC ? lcol * BK + (((2 * pr + lrow) ^ kc_swizzle(lcol)) * 4) : (8 * pr + 4 * lrow) * BM + lcol;
        offb[pr] = BKC ? lcol * BK + (((2 * pr + lrow) ^ kc_swizzle(lcol)) * 4) : (8 * pr + 4 * lrow) * BN + lcol;
    }
    float raw[BLOCKS][8];
    auto read_block = [&](auto blkc, float (&x)[8], int stage) {
        constexpr int blk = decltype(blkc)::value, r = blk < 2 ? blk : blk - 2;
        constexpr bool KC = blk < 2 ? AKC : BKC;
        const float* s = &S[kg][0] + (blk < 2 ? stage * TILE_A : NST * TILE_A + stage * TILE_B);
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
            const float* q = s + (blk < 2 ? offa[pr] : offb[pr]) + r * (KC ? 32 * BK : 32);
            if (KC) {
                const float4 v = *reinterpret_cast<const float4*>(q);
                x[4 * pr] = v.x; x[4 * pr + 1] = v.y; x[4 * pr + 2] = v.z; x[4 * pr + 3] = v.w;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) x[4 * pr + c] = q[c * (blk < 2 ? BM : BN)];
            }
        }
    };
    constexpr bool SA = !(AKC && BKC), SB = !AKC && !BKC;
    const float scale_a = SA ? p.scale_a : 1.f, scale_b = SB ? p.scale_b : 1.f;
    uint32_t hp[2][BLOCKS][4], lp[2][BLOCKS][4];
    // the i-th of the 12 BLOCKS pieces of a k-tile's split: block by block, each step for all four pairs
    auto split_piece = [&](auto ic, auto setc) {
        constexpr int i = decltype(ic)::value, set = decltype(setc)::value, blk = i / 12, st = i / 4 % 3, j = i % 4;
        split_step<st, (blk < 2 ? SA : SB)>(raw[blk][2 * j], raw[blk][2 * j + 1], hp[set][blk][j], lp[set][blk][j], blk < 2 ? scale_a : scale_b);
    };
    floatx16 acc[SETS][PRODUCTS], low[PRODUCTS];
    static_for<PRODUCTS>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        acc[0][q] = acc[SETS - 1][q] = low[q] = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    });
    auto part = [](const uint32_t (&x)[4]) { return __builtin_bit_cast(halfx8, uintx4{x[0], x[1], x[2], x[3]}); };
    auto mfma = [&](auto qc, auto setc) {
        constexpr int set = decltype(setc)::value, pr = decltype(qc)::value / PRODUCTS, q = decltype(qc)::value % PRODUCTS, i = q / TN, j = 2 + q % TN, at = set % SETS;
        if constexpr (pr == 0) low[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(part(lp[set][i]), part(hp[set][j]), low[q], 0, 0, 0);
        else if constexpr (pr == 1) acc[at][q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(part(hp[set][i]), part(hp[set][j]), acc[at][q], 0, 0, 0);
        else low[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(part(hp[set][i]), part(lp[set][j]), low[q], 0, 0, 0);
    };

    // Contraction steps past the last whole k-tile: the last k-group's, requested ahead of every direct load (see gemm_dma_kg_body), or behind
    // the loop where it leaves no registers for them.
    const bool has_tail = kg == KG - 1 && ktail < kend;
    float tail[BLOCKS][8];
    auto request_tail = [&]() {
        if (!has_tail) return;
        const float* __restrict__ Ab = p.A + (int64_t)b * p.a_bstride;
        const float* __restrict__ Bb = p.B + (int64_t)b * p.b_bstride;
        static_for<BLOCKS>([&](auto blkc) {
            constexpr int blk = decltype(blkc)::value;
            const int m = min(m0 + 32 * blk + lcol, p.M - 1), n = min(n0 + 32 * (blk - 2) + lcol, p.N - 1);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int k = ktail + 8 * (c / 4) + 4 * lrow + c % 4;
                if constexpr (blk < 2) tail[blk][c] = k < p.K ? (AKC ? Ab[(int64_t)m * p.lda + k] : Ab[(int64_t)k * p.lda + m]) : 0.f;
                else tail[blk][c] = k < p.K ? (BKC ? Bb[(int64_t)n * p.ldb + k] : Bb[(int64_t)k * p.ldb + n]) : 0.f;
            }
        });
    };
    if constexpr (TN == 2) request_tail();
#pragma unroll
    for (int t = 0; t < NST; ++t)
        if (t < nkt) issue(t, t);
    typedef std::integral_constant<int, 0> C0;
    if (nkt >= NST) wait_kg64<(NST - 1) * LOADS>();
    else wait_kg64<0>();
    static_for<BLOCKS>([&](auto blkc) { read_block(blkc, raw[decltype(blkc)::value], 0); });
    // (which operands take the fp32 MFMAs: as in gemm_dma_kg_body)
    bool any = p.three != 0;
    static_for<BLOCKS>([&](auto blkc) {
        constexpr int blk = decltype(blkc)::value;
        float most = 0.f;
        static_for<4>([&](auto jc) { most_of(most, raw[blk][2 * decltype(jc)::value], raw[blk][2 * decltype(jc)::value + 1]); });
        most *= blk < 2 ? scale_a : scale_b;
        any |= !(most >= (blk < 2 ? p.least_a : kSplitLeast) && most < kSplitMost);
    });
    const bool plain = __any(any);
    if (__builtin_expect(plain, 0)) {
        for (int t = 0; t < nkt; ++t) {
            static_for<8>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                static_for<PRODUCTS>([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
                    floatx16& to = c % 2 ? low[q] : acc[0][q];
                    to = __builtin_amdgcn_mfma_f32_32x32x2f32(raw[q / TN][c] * scale_a, raw[2 + q % TN][c] * scale_b, to, 0, 0, 0);
                });
            });
            __builtin_amdgcn_sched_barrier(0);      // (tile t's reads are behind it)
            if (t + 1 < nkt) {
                if (t + NST < nkt) { issue(t + NST, t % NST); wait_kg64<(NST - 1) * LOADS>(); }
                else wait_kg64<0>();
                const int stage = (t + 1) % NST;
                static_for<BLOCKS>([&](auto blkc) { read_block(blkc, raw[decltype(blkc)::value], stage); });
            }
        }
    } else {
        static_for<12 * BLOCKS>([&](auto ic) { split_piece(ic, C0{}); });
        if (nkt >= NST) wait_kg64<(NST - 2) * LOADS>();
        if (nkt > 1) static_for<BLOCKS>([&](auto blkc) { read_block(blkc, raw[decltype(blkc)::value], 1); });
        __builtin_amdgcn_sched_barrier(0);
        auto step = [&](auto uc, const int t) {
            constexpr int u = decltype(uc)::value, set = u & 1;
            typedef std::integral_constant<int, set> Set;
            typedef std::integral_constant<int, set ^ 1> Next;
            if (t + NST < nkt) issue(t + NST, u % NST);      // (tile t's reads are behind its split)
            __builtin_amdgcn_sched_barrier(0);
            constexpr int MFMAS = 3 * PRODUCTS, PIECES = 12 * BLOCKS / MFMAS;
            static_assert(PIECES * MFMAS == 12 * BLOCKS, "as many pieces behind every MFMA");
            static_for<MFMAS>([&](auto qc) {
                constexpr int q = decltype(qc)::value, rd = q - (MFMAS - BLOCKS);
                mfma(qc, Set{});
                static_for<PIECES>([&](auto sc) { split_piece(std::integral_constant<int, PIECES * q + decltype(sc)::value>{}, Next{}); });
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (rd == -1) {
                    if (t + NST < nkt) wait_kg64<(NST - 2) * LOADS>();
                    else wait_kg64<0>();
                }
                if constexpr (rd >= 0) {
                    // (behind the last tiles: what an earlier one left there, and nobody uses)
                    read_block(std::integral_constant<int, rd>{}, raw[rd], (u + 2) % NST);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };
        constexpr int PERIOD = NST % 2 ? 2 * NST : NST;
        for (int t = 0; t < nkt; t += PERIOD)
            static_for<PERIOD>([&](auto uc) { if (t + decltype(uc)::value < nkt) step(uc, t + decltype(uc)::value); });
    }
    const float unscale = power_of_two_over(scale_a, 0) * power_of_two_over(scale_b, 0);
    const float low_scale = plain ? 1.f : 0x1p-11f;
    if constexpr (TN == 4) request_tail();
    float* park = &S[kg][0];
    static_for<PRODUCTS>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        floatx16 s;
        static_for<16>([&](auto vc) {
            constexpr int v = decltype(vc)::value;
            s[v] = __builtin_fmaf(low[q][v], low_scale, SETS == 2 ? acc[0][q][v] + acc[SETS - 1][q][v] : acc[0][q][v]);
            if constexpr (SA || SB) s[v] *= unscale;
        });
        if (block_suspect(s)) {
            const float *Ab = p.A + (int64_t)b * p.a_bstride, *Bb = p.B + (int64_t)b * p.b_bstride;
            s = block_fp32<AKC, BKC>(Ab, p.lda, Bb, p.ldb, p.M, p.N, m0 + 32 * (q / TN), n0 + 32 * (q % TN), kbeg, kbeg + ((nkt - 1) * KG + 1) * BK, KG * BK / kSplitBK);
        }
        if (has_tail)
            static_for<8>([&](auto cc) { s = __builtin_amdgcn_mfma_f32_32x32x2f32(tail[q / TN][decltype(cc)::value], tail[2 + q % TN][decltype(cc)::value], s, 0, 0, 0); });
        static_for<16>([&](auto vc) { constexpr int v = decltype(vc)::value; park[q * 1024 + v * 64 + lane] = s[v]; });
    });
    // The k-groups' sums in group order, wavefront g adds up and writes TN / 2 neighbouring blocks.
    __syncthreads();
    constexpr int MINE = TN / 2;
    floatx16 sum[1][MINE];
    static_for<MINE * 16>([&](auto vc) {
        constexpr int e = decltype(vc)::value / 16, v = decltype(vc)::value % 16;
        const int at = (kg * MINE + e) * 1024 + v * 64 + lane;
        float r = S[0][at];
#pragma unroll
        for (int g = 1; g < KG; ++g) r += S[g][at];
        sum[0][e][v] = r;
    });
    const int mb = m0 + 32 * (kg * MINE / TN), nb = n0 + 32 * (kg * MINE % TN);
    if (p.splits > 1) {
        Epilogue raw{};
        EpiCtx c{};
        c.alpha = 1.f;
        c.C = p.ws + ((int64_t)bz * p.M) * p.N;
        write_tile<EPI_STORE, 1, MINE>(sum, raw, c, p.N, p.M, p.N, mb, nb, lrow, lcol);
        return;
    }
    const EpiCtx c = epi_ctx(p.epi, p.C, p.c_bstride, b);
    MAVG_EPI_DISPATCH(p.epi.kind, (write_tile<KIND, 1, MINE>(sum, p.epi, c, p.ldc, p.M, p.N, mb, nb, lrow, lcol)))
}

}  // namespace mavg
