// Device side of the fp32 GEMM on the bf16 matrix cores: every fp32 operand element is split exactly into three
// bf16 parts (8 + 8 + 8 significant bits) and the six products of parts that matter in fp32 are accumulated in fp32.
//
// Why: v_mfma_f32_32x32x2_f32 runs at 157 TFLOP/s, v_mfma_f32_32x32x16_bf16 at 2.2 - 2.4 PFLOP/s (measured, with and
// without vector work beside it; 1.6 - 1.8 with operands of random bits, where the chip lowers its clock).  Six bf16
// products per fp32 product still leave 370 (270 - 300) TFLOP/s.
//
// What bounds it (128x128 tiles, 4096^3): 190 TFLOP/s on random values, 264 on zeros - the power limit; before, with fp32
// MFMAs, 149.  On fewer tiles than fill the chip: LDS, which takes the three parts at 64 bytes per cycle (ds_write of any
// width; reads run at 240), beside the reads and the matrix pipe: 1024 x 2048 x 2048 60 us, was 66 - 80.
//
// What it computes.  x = h + m + l with h = bf16(x) and m = bf16(x - h), rounded to nearest, and l = the rest; the split is
// exact for |x| >= 2^-110 and off by at most 2^-133 below that.  Products of bf16 values are exact in fp32, and the matrix
// cores add eight of them to the accumulator with one rounding to nearest (measured; denormals are kept).  h h', h m', m h',
// m m', h l', l h' are accumulated; m l', l m' and l l' are left out: for |x| in [1, 2), |m| <= 2^-8 and |l| <= 2^-17, so
// together at most 2^-24 of |x x'| (1 + 2^-9), the largest rounding of an fp32 product, and 2^-28.2 in the mean with either
// sign (2^-25.5 for the rounding of an fp32 product).  A truncated m would leave |l| up to 2^-16 and twice to three times
// that: 2^-23 at most, 2^-26.7 in the mean.
// Against float64 the results are as close as those of the fp32 matrix cores (12 roundings of the accumulator per 16
// contraction steps here, 16 there).
//
// Infinities, NaNs and values that round to infinity in bf16 (above 3.39e38) do not survive the split (inf - inf, and
// inf * 0 where a part of the other factor is zero).  They always leave a NaN or an infinity in the accumulators they
// reach, so a wavefront that finds a non-finite accumulator recomputes that 32x32 block with the fp32 matrix cores:
// what is returned is then what fp32 arithmetic gives.  Microseconds for ordinary values, one infinity and nothing but NaNs:
// 1024 x 2048 x 2048 60 / 94 / 174 (fp32 kernels alone 68; with single loads in the recomputation 60 / 151 / 488),
// 4096 x 8000 x 2048 712 / 816 / 2385 (fp32 920; with single loads 758 / 991 / 7654).
//
// Small values.  An element below 2^-110 loses up to 2^-133 in the split, so a sum over terms x x' may be off by
// 2^-133 times the sum of the other factors' magnitudes.  Where that could matter the sum itself is small: a block with an
// accumulator below 2^-80 other than zero is recomputed as well.  What is left is 2^-53 of a result times the sum of the other
// factors' magnitudes (below 2^-24 unless those come to 2^29), and blocks whose sums are all zero because no element of an
// operand reaches 2^-134.  (Recomputing blocks of zeros too: a CD-1 step of 822 rows, 918 x 242, 152 us instead of 142.  Scaling
// every element by 2^16 before its split would keep them all, at 6 - 9 % of every product; this takes 0 - 4 %.)
#pragma once
#include "gemm_device.h"

namespace mavg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));     // a 16-byte load from a 4-byte aligned address
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) float* GlobalF;             // global memory, not "any address space"
typedef const __attribute__((address_space(1))) floatx4u* GlobalF4;
__device__ __forceinline__ GlobalF g_off(GlobalF ubase, uint32_t off) {      // scalar base + 32-bit lane offset
    return (GlobalF)((const __attribute__((address_space(1))) char*)ubase + (uint64_t)off);
}

// Two floats -> their three parts, packed (h, m, l), in three steps of three or four vector instructions, so that they can
// be dealt out between matrix instructions; x0, x1 hold the remainders on the way (all differences are exact).  Ordinary
// vector instructions issue beside the matrix pipe (six of them per MFMA cost it nothing: 34 cycles per MFMA measured).
// v_dot2_f32_bf16, which unpacks and subtracts at once, does not: two of them per MFMA make it 62 cycles.
template <int STEP>
__device__ __forceinline__ void split_step(float& x0, float& x1, uint32_t& h, uint32_t& m, uint32_t& l, const uint32_t kHigh) {
    constexpr uint32_t kPackHigh = 0x07060302u;
    // (an instruction of its own: from the C conversions the compiler makes a second one for the low half)
    auto round_pair = [&](uint32_t& d) { asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(d) : "v"(x0), "v"(x1)); };
    if constexpr (STEP == 0) {
        round_pair(h);
        x0 -= __builtin_bit_cast(float, h << 16);
        l = h & kHigh;
    } else if constexpr (STEP == 1) {
        x1 -= __builtin_bit_cast(float, l);
        round_pair(m);
        x0 -= __builtin_bit_cast(float, m << 16);
    } else {
        x1 -= __builtin_bit_cast(float, m & kHigh);
        l = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, x1), __builtin_bit_cast(uint32_t, x0), kPackHigh);
    }
}

// Does the wavefront's 32x32 block hold an infinity or a NaN (x * 0 is NaN exactly then), or a value below 2^-80 other than
// zero?  (First the least magnitude with the zeros among it: one and a half instructions per element.)
__device__ __forceinline__ bool block_suspect(const floatx16& a) {
    constexpr float kTiny = 0x1p-80f;
    float t = 0.f, least = 1.f;
    static_for<16>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        t = __builtin_fmaf(a[v], 0.f, t);
        least = fminf(least, fabsf(a[v]));
    });
    asm("" : "+v"(least));      // (a minimum, not a comparison per element)
    bool odd = !(t == 0.f);
    if (!__any(odd || least < kTiny)) return false;
    static_for<16>([&](auto vc) {
        const float x = fabsf(a[decltype(vc)::value]);
        odd |= x < kTiny && x != 0.f;
    });
    return __any(odd);
}

constexpr int kSplitBK = 16;      // contraction steps per k-tile: one MFMA

// The 32x32 block at (mb, nb) over contraction steps [kbeg, kend), of which those of every `stride`-th k-tile, on the fp32
// matrix cores.  Lane half `lrow` multiplies steps 8 lrow .. 8 lrow + 7 of a k-tile, which it reads from a k-contiguous
// operand with two 16-byte loads (single floats touch four times the cache lines, and those are what bounds this); a k-tile
// is on its way while the one before is multiplied.
template <bool AKC, bool BKC>
__device__ __forceinline__ floatx16 block_fp32(const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N,
                                               int mb, int nb, int kbeg, int kend, int stride) {
    const int lane = threadIdx.x & 63, lrow = lane >> 5, lcol = lane & 31, hop = stride * kSplitBK;
    const GlobalF ra = (GlobalF)(A + (int64_t)min(mb + lcol, M - 1) * (AKC ? lda : 1));      // this lane's row (or column)
    const GlobalF rb = (GlobalF)(B + (int64_t)min(nb + lcol, N - 1) * (BKC ? ldb : 1));
    auto fetch = [&](GlobalF p, int64_t ld, auto kcc, int kt, float (&x)[8]) {
        constexpr bool KC = decltype(kcc)::value;
        const int k = kt + 8 * lrow;
        if (kt + kSplitBK <= kend) {      // (uniform)
            if constexpr (KC) {
                const floatx4u u = *(GlobalF4)(p + k), v = *(GlobalF4)(p + k + 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) { x[i] = u[i]; x[4 + i] = v[i]; }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = p[(int64_t)(k + i) * ld];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                x[i] = 0.f;
                if (k + i < kend) x[i] = p[KC ? (int64_t)(k + i) : (int64_t)(k + i) * ld];
            }
        }
    };
    floatx16 acc = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float a[8], b[8], an[8] = {}, bn[8] = {};
    if (kbeg < kend) {
        fetch(ra, lda, std::integral_constant<bool, AKC>{}, kbeg, a);
        fetch(rb, ldb, std::integral_constant<bool, BKC>{}, kbeg, b);
    }
#pragma unroll 1
    for (int kt = kbeg; kt < kend; kt += hop) {
        if (kt + hop < kend) {
            fetch(ra, lda, std::integral_constant<bool, AKC>{}, kt + hop, an);
            fetch(rb, ldb, std::integral_constant<bool, BKC>{}, kt + hop, bn);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) { a[i] = an[i]; b[i] = bn[i]; }
    }
    return acc;
}

// One operand's share of a k-tile in a thread's registers: units of W contraction steps of one row.
//   k-contiguous operand: W = 4, unit c -> row c / 4, steps 4 (c % 4) ..: four neighbouring lanes read the 64 bytes of one
//     row with one load (two lanes of 8 steps each, two loads apiece, touch twice the cache lines per load)
//   m/n-contiguous operand: W = 8, unit c -> row c % BR, steps 8 (c / BR) ..: a wavefront reads 256 bytes of each of 8 k-rows
template <int BR, int NT, bool KC>
struct SplitOperand {
    static constexpr int BK = kSplitBK, W = KC ? 4 : 8, Q = BK / W, CH = BR * Q / NT;     // units per row, units per thread
    static_assert(CH >= 1 && CH * NT == BR * Q, "tile does not divide over the threads");
    static_assert(KC || NT % BR == 0 || BR % NT == 0, "rows of a thread's units");
    // LDS: [plane][8-step half][row] of 16 bytes.  Reads (32 rows of one half) and the writes of an m/n-contiguous operand run
    // over consecutive rows; the writes of a k-contiguous operand cover both halves of 16 rows, which the swizzle of the
    // second half keeps on different banks.
    static constexpr int QS = BR * 16, PS = 2 * QS, STAGE = 3 * PS;     // bytes
    static __device__ __forceinline__ int place(int r, int half) { return half * QS + (KC ? r ^ (8 * half) : r) * 16; }
    uint32_t off[CH];       // this lane's byte offset inside the operand's tile, per unit
    uint32_t dst[CH];       // ... and inside an LDS plane
    GlobalF base;           // (uniform) row r0 (or column), contraction step kfull
    int64_t ld;

    // kfull: where the first whole k-tile begins
    __device__ __forceinline__ void init(const float* P, int64_t ld_, int r0, int R, int64_t kfull, int tid) {
        ld = (int64_t)uniform_u64((uint64_t)ld_);
        base = (GlobalF)uniform_u64(reinterpret_cast<uint64_t>(KC ? P + (int64_t)r0 * ld_ + kfull : P + kfull * ld_ + r0));
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = tid + i * NT;
            const int r = KC ? c / Q : c % BR, q = KC ? c % Q : c / BR;
            const int row = min(r, R - 1 - r0);                 // rows past the edge repeat the last one (never stored)
            off[i] = KC ? (uint32_t)(((int64_t)row * ld_ + W * q) * 4) : (uint32_t)((W * q * ld_ + row) * 4);
            dst[i] = (uint32_t)(KC ? place(r, q >> 1) + 8 * (q & 1) : place(r, q));
        }
    }
    // the units of the contraction steps from step `k` on: a whole k-tile (FULL), or one of `left` steps (zeros past them)
    template <bool FULL>
    __device__ __forceinline__ void load(int k, int left, float (&x)[CH][W], int tid) const {
        const GlobalF b = base + (KC ? (int64_t)k : (int64_t)k * ld);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if constexpr (!FULL) {
                const int c = tid + i * NT, q = KC ? c % Q : c / BR;
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    x[i][j] = 0.f;
                    if (W * q + j < left) x[i][j] = *g_off(KC ? b + j : b + j * ld, off[i]);
                }
            } else if constexpr (KC) {
                const floatx4u u = *(GlobalF4)g_off(b, off[i]);
#pragma unroll
                for (int j = 0; j < 4; ++j) x[i][j] = u[j];
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] = *g_off(b + j * ld, off[i]);
            }
        }
    }
    // The split of a thread's units into LDS planes, in PIECES steps (W / 2 pairs of three steps per unit).
    static constexpr int PER = W / 2 * 3, PIECES = CH * PER;
    template <int I>
    __device__ __forceinline__ void piece(char* S, float (&x)[CH][W], uint32_t (&h)[4], uint32_t (&m)[4], uint32_t (&l)[4], uint32_t high) const {
        constexpr int i = I / PER, j = I % PER / 3, st = I % 3;
        split_step<st>(x[i][2 * j], x[i][2 * j + 1], h[j], m[j], l[j], high);
        if constexpr (I % PER == PER - 1) {
            if constexpr (KC) {
                *reinterpret_cast<uintx2*>(S + dst[i]) = uintx2{h[0], h[1]};
                *reinterpret_cast<uintx2*>(S + dst[i] + PS) = uintx2{m[0], m[1]};
                *reinterpret_cast<uintx2*>(S + dst[i] + 2 * PS) = uintx2{l[0], l[1]};
            } else {
                *reinterpret_cast<uintx4*>(S + dst[i]) = uintx4{h[0], h[1], h[2], h[3]};
                *reinterpret_cast<uintx4*>(S + dst[i] + PS) = uintx4{m[0], m[1], m[2], m[3]};
                *reinterpret_cast<uintx4*>(S + dst[i] + 2 * PS) = uintx4{l[0], l[1], l[2], l[3]};
            }
        }
    }
};

// BM x BN output tile by KG groups of WM x WN wavefronts, each wavefront owning (BM/WM) x (BN/WN) as TM x TN accumulators
// of 32x32.  The k-groups take a share of the contraction range each, with LDS buffers of their own, and add their
// accumulators through LDS at the end (in group order): more wavefronts per tile where tiles are few.
// Pipeline: while tile t is multiplied, a later one is split into the LDS buffer that is free and the two after that are on
// their way into registers; one barrier per k-tile.
template <int BM, int BN, int WM, int WN, int KG, bool AKC, bool BKC>
__device__ __forceinline__ void gemm_split_body(const GemmKParams& p, const int tile, const int bz) {
    constexpr int BK = kSplitBK;
    constexpr int NT = 64 * WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    using OpA = SplitOperand<BM, NT, AKC>;
    using OpB = SplitOperand<BN, NT, BKC>;
    constexpr int STAGE = OpA::STAGE + OpB::STAGE;
    constexpr int PARK = KG > 1 ? BM * BN * 4 : 0;       // a k-group's accumulators, for the final sum
    __shared__ __attribute__((aligned(1024))) char Sall[KG * (2 * STAGE > PARK ? 2 * STAGE : PARK)];

    const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int tid = (int)threadIdx.x - kg * NT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char* S = Sall + kg * 2 * STAGE;
    const int lrow = lane >> 5, lcol = lane & 31;
    const int wm = (wave / WN) * (32 * TM), wn = (wave % WN) * (32 * TN);
    const int b = bz / p.splits, split = bz - b * p.splits;
    int tm_i, tn_i;
    tile_coords(p, tile, tm_i, tn_i);
    const int m0 = tm_i * BM, n0 = tn_i * BN;
    const int kbeg = split * p.kper, kend = min(p.K, kbeg + p.kper);
    // k-group g takes k-tiles g, g + KG, ...: what the groups of a workgroup read at a time are neighbouring pieces of the
    // same cache lines (a k-tile is half a line of a k-contiguous operand): 1024 x 2048 x 2048 55.9 against 59.1 us with a
    // contiguous share per group, 256 x 8000 x 2048 57.0 against 64.8.
    constexpr int KS = KG * BK;
    const int all = (kend - kbeg + BK - 1) / BK, first = kbeg + kg * BK;
    const int nloop = (all + KG - 1) / KG;                     // every wavefront takes part in this many barriers
    const int nkt = __builtin_amdgcn_readfirstlane(all > kg ? (all - kg + KG - 1) / KG : 0);
    const float* A = p.A + (int64_t)b * p.a_bstride;
    const float* B = p.B + (int64_t)b * p.b_bstride;
    OpA oa;
    OpB ob;
    // A partial k-tile (contraction not a multiple of 16) goes first, so that the loop's loads are all whole ones and
    // their number in flight is known: tile 0 is the last `left` steps then, tile t > 0 the (t - 1)-th whole one.
    // (The host sends contractions of at least 16 steps.  A group without a whole tile reads, and never uses, the first
    // whole one of the range, or the one before a range that is a partial tile alone, which is not the first range.)
    const int left = nkt > 0 && (all - 1) % KG == kg ? (kend - kbeg) % BK : 0, part = left > 0 ? 1 : 0;
    const int kwhole = nkt > part ? first : kend - kbeg >= BK ? kbeg : kbeg - BK;
    oa.init(A, p.lda, m0, p.M, kwhole, tid);
    ob.init(B, p.ldb, n0, p.N, kwhole, tid);

    floatx16 acc[TM][TN];
    static_for<TM * TN>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        acc[t / TN][t % TN] = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    });
    // Fused (optionally weighted) row sums of A, by the workgroups of the first tile column, from the fp32 elements a
    // thread has in registers: thread group rs_grp sums its chunks of row rs_row, the groups' sums meet in LDS after
    // the loop.  The weights are uniform over the wavefront and come by scalar loads.
    constexpr int RS_G = NT / BM > 0 ? NT / BM : 1;
    const bool rs_block = !AKC && KG == 1 && NT % BM == 0 && p.epi.rowsum_dst != nullptr && tn_i == 0;
    const int rs_grp = __builtin_amdgcn_readfirstlane(tid / BM), rs_row = tid % BM;
    float rowsum = 0.f;
    typedef const __attribute__((address_space(4))) float* ConstF;
    const ConstF rw = p.epi.rowsum_w
        ? (ConstF)reinterpret_cast<uintptr_t>(p.epi.rowsum_w + (int64_t)b * p.epi.rowsum_w_bstride + kbeg) : (ConstF)0;

    float xa[2][OpA::CH][OpA::W], xb[2][OpB::CH][OpB::W];       // two k-tiles on their way, tile t in set t & 1
    auto load = [&](int tl, auto setc) {
        const int k = max(min(tl, nkt - 1) - part, 0) * KS;
        oa.template load<true>(k, BK, xa[decltype(setc)::value], tid);
        ob.template load<true>(k, BK, xb[decltype(setc)::value], tid);
    };
    auto row_sums = [&](int t, auto setc) {
        constexpr int set = decltype(setc)::value;
        if constexpr (!AKC) {
            if (!rs_block || t >= nkt) return;
#pragma unroll
            for (int i = 0; i < OpA::CH; ++i) {
                const int q = rs_grp + i * RS_G;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = (t < part ? kend - left - kbeg : (t - part) * KS) + 8 * q + j;      // (one k-group: from kbeg on)
                    if (rw) { if (k < kend - kbeg) rowsum += xa[set][i][j] * rw[k]; }
                    else rowsum += xa[set][i][j];
                }
            }
        }
    };
    // step I of the split of the k-tile in register set `setc` into the LDS buffer of the same number
    uint32_t ph[4], pm[4], pl[4];
    uint32_t high = 0xffff0000u;      // in a scalar register: half the instruction bytes of a literal
    asm volatile("" : "+s"(high));
    constexpr int PIECES = OpA::PIECES + OpB::PIECES;
    auto piece = [&](auto ic, auto setc) {
        constexpr int I = decltype(ic)::value, set = decltype(setc)::value;
        if constexpr (I < OpA::PIECES) oa.template piece<I>(S + set * STAGE, xa[set], ph, pm, pl, high);
        else ob.template piece<I - OpA::PIECES>(S + set * STAGE + OpA::STAGE, xb[set], ph, pm, pl, high);
    };
    auto stage = [&](auto setc) { static_for<PIECES>([&](auto ic) { piece(ic, setc); }); };
    const char* fa_base = S + OpA::place(wm + lcol, lrow);
    const char* fb_base = S + OpA::STAGE + OpB::place(wn + lcol, lrow);
    // With four accumulators per wavefront a second operand set does not fit the 256 registers that two wavefronts per SIMD
    // leave each other: a step then begins with its own reads (and the other workgroup's MFMAs cover them).
    constexpr bool PRE = TM * TN < 4;
    constexpr int LEAD = PRE ? 2 : 1;          // the tile that step t splits is t + LEAD
    bf16x8 fa[PRE ? 2 : 1][3][TM], fb[PRE ? 2 : 1][3][TN];
    constexpr int READS = 3 * (TM + TN);
    // read number I of the MFMA operands of the k-tile in LDS buffer `bufc` (into the operand set of the same number)
    auto read_frag = [&](auto ic, auto bufc) {
        constexpr int I = decltype(ic)::value, buf = decltype(bufc)::value, pl = I / (TM + TN), r = I % (TM + TN);
        constexpr int fs = PRE ? buf : 0;
        if constexpr (r < TM) fa[fs][pl][r] = *reinterpret_cast<const bf16x8*>(fa_base + buf * STAGE + pl * OpA::PS + r * 512);
        else fb[fs][pl][r - TM] = *reinterpret_cast<const bf16x8*>(fb_base + buf * STAGE + pl * OpB::PS + (r - TM) * 512);
    };
    // A wavefront that is a k-group by itself needs no s_barrier: its LDS instructions are carried out in order.  The fences
    // keep the compiler from moving an LDS access across, which another lane's data may depend on.
    auto group_barrier = [&]() {
        if constexpr (NT > 64) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    };
    // One k-tile t.  Behind each of its MFMAs goes a share of the other work, which issues while the matrix pipe works:
    //   PRE: the operand reads of tile t+1 (LDS buffer (t+1) & 1) and the split of tile t+2 into LDS buffer t & 1, whose
    //        reads every wavefront had finished before the last barrier;
    //   otherwise: the split of tile t+1 into LDS buffer (t+1) & 1 (likewise).
    auto step = [&](auto parc) {
        constexpr int par = decltype(parc)::value, set = PRE ? par : par ^ 1, fs = PRE ? par : 0;
        constexpr int NMF = 6 * TM * TN;
        if constexpr (!PRE) {
            static_for<READS>([&](auto ic) { read_frag(ic, parc); });
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<NMF>([&](auto qc) {
            constexpr int q = decltype(qc)::value, pr = q / (TM * TN), i = q / TN % TM, j = q % TN;
            constexpr int pa = pr == 1 || pr == 3 ? 1 : pr == 5 ? 2 : 0;      // hh, mh, hm, mm, hl, lh
            constexpr int pb = pr == 2 || pr == 3 ? 1 : pr == 4 ? 2 : 0;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[fs][pa][i], fb[fs][pb][j], acc[i][j], 0, 0, 0);
            if constexpr (PRE) {
                constexpr int r0 = q * READS / NMF, r1 = (q + 1) * READS / NMF;
                static_for<r1 - r0>([&](auto ic) { read_frag(std::integral_constant<int, r0 + decltype(ic)::value>{}, std::integral_constant<int, par ^ 1>{}); });
            }
            constexpr int p0 = q * PIECES / NMF, p1 = (q + 1) * PIECES / NMF;
            static_for<p1 - p0>([&](auto ic) { piece(std::integral_constant<int, p0 + decltype(ic)::value>{}, std::integral_constant<int, set>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, 1> C1;
    if (left > 0) {
        oa.template load<false>(kend - left - kwhole, left, xa[0], tid);
        ob.template load<false>(kend - left - kwhole, left, xb[0], tid);
    } else {
        load(0, C0{});
    }
    load(1, C1{});
    row_sums(0, C0{});
    stage(C0{});
    load(2, C0{});
    if constexpr (PRE) {
        row_sums(1, C1{});
        stage(C1{});
        load(3, C1{});
        group_barrier();
        static_for<READS>([&](auto ic) { read_frag(ic, C0{}); });
    }
    group_barrier();
    // (The last steps load the last tile again and split it into buffers nobody reads: unconditional loads keep the
    // number in flight known, and one loop without special cases keeps the accumulators where they are.)
    typedef std::integral_constant<int, PRE ? 0 : 1> Even;      // the register set that step t = 0, 2, ... empties and refills
    typedef std::integral_constant<int, PRE ? 1 : 0> Odd;
    for (int t = 0; t < nkt; t += 2) {
        row_sums(t + LEAD, Even{});
        step(C0{});
        load(t + LEAD + 2, Even{});
        group_barrier();
        if (t + 1 >= nkt) break;
        row_sums(t + LEAD + 1, Odd{});
        step(C1{});
        load(t + LEAD + 3, Odd{});
        group_barrier();
    }
    if constexpr (KG > 1)
        for (int i = nkt; i < nloop; ++i) group_barrier();

    static_for<TM * TN>([&](auto tc) {
        constexpr int i = decltype(tc)::value / TN, j = decltype(tc)::value % TN;
        if (block_suspect(acc[i][j]))
            acc[i][j] = block_fp32<AKC, BKC>(A, p.lda, B, p.ldb, p.M, p.N, m0 + wm + 32 * i, n0 + wn + 32 * j, first, kend, KG);
    });

    int bands = -1;
    if constexpr (KG > 1) {
        // Each wavefront parks its accumulators; k-group g then adds up bands g of 16 / KG elements each and writes those.
        float* red = reinterpret_cast<float*>(Sall);
        constexpr int W = WM * WN, V = TM * TN * 16, PER = KG > 4 ? 1 : 4 / KG;
        static_assert(KG == 2 || KG == 4 || KG == 8, "four bands of four elements to share out");
        if constexpr (NT == 64) __syncthreads();
        static_for<TM * TN>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            static_for<16>([&](auto vc) {
                constexpr int v = decltype(vc)::value;
                red[((kg * W + wave) * V + t * 16 + v) * 64 + lane] = acc[t / TN][t % TN][v];
            });
        });
        __syncthreads();
        bands = kg * PER < 4 ? ((1 << PER) - 1) << (kg * PER) : 0;
        static_for<TM * TN>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            static_for<16>([&](auto vc) {
                constexpr int v = decltype(vc)::value;
                if ((bands >> (v >> 2)) & 1) {
                    float r = red[(wave * V + t * 16 + v) * 64 + lane];
#pragma unroll
                    for (int g = 1; g < KG; ++g) r += red[((g * W + wave) * V + t * 16 + v) * 64 + lane];
                    acc[t / TN][t % TN][v] = r;
                }
            });
        });
    }
    if (rs_block) {       // (workgroup-uniform) the groups' partial sums, added in the order of the groups
        float* red = reinterpret_cast<float*>(S);
        if (rs_grp > 0) red[(rs_grp - 1) * BM + rs_row] = rowsum;
        __syncthreads();
        if (rs_grp == 0) {
#pragma unroll
            for (int g = 1; g < RS_G; ++g) rowsum += red[(g - 1) * BM + rs_row];
            if (m0 + rs_row < p.M) {
                float* d = p.epi.rowsum_dst + (int64_t)b * p.epi.rowsum_bstride + m0 + rs_row;
                float r = p.epi.rowsum_alpha * rowsum;
                if (p.epi.alpha_dev0) r *= p.epi.alpha_dev0[b];
                if (p.epi.alpha_dev1) r *= p.epi.alpha_dev1[b];
                if (p.epi.rowsum_beta != 0.f) r += p.epi.rowsum_beta * *d;
                *d = r;
                if (p.epi.rowsum_dst2) p.epi.rowsum_dst2[(int64_t)b * p.epi.rowsum2_bstride + m0 + rs_row] += r;
            }
        }
    }
    if (p.splits > 1) {
        Epilogue raw;
        EpiCtx c;
        c.bias = nullptr; c.aux = nullptr; c.C2 = nullptr; c.rowvec = nullptr; c.alpha = 1.f; c.lastcol_dst = nullptr;
        c.C = p.ws + ((int64_t)bz * p.M) * p.N;
        write_tile<EPI_STORE, TM, TN>(acc, raw, c, p.N, p.M, p.N, m0 + wm, n0 + wn, lrow, lcol, bands);
    } else {
        const EpiCtx c = epi_ctx(p.epi, p.C, p.c_bstride, b);
        MAVG_EPI_DISPATCH(p.epi.kind, (write_tile<KIND, TM, TN>(acc, p.epi, c, p.ldc, p.M, p.N, m0 + wm, n0 + wn, lrow, lcol, bands)))
    }
}

template <int BM, int BN, int WM, int WN, int KG, int OCC, bool AKC, bool BKC>
__global__ __launch_bounds__(64 * WM * WN * KG, OCC) void gemm_split_kernel(GemmKParams p) {
    gemm_split_body<BM, BN, WM, WN, KG, AKC, BKC>(p, blockIdx.x, blockIdx.z);
}

template <int BM, int BN, int WM, int WN, int KG, int OCC, bool AKC, bool BKC>
__global__ __launch_bounds__(64 * WM * WN * KG, OCC) void gemm_split_grouped_kernel(GemmGroupParams gp) {
    int first;
    const GemmKParams& p = group_params(gp, first);
    gemm_split_body<BM, BN, WM, WN, KG, AKC, BKC>(p, (int)blockIdx.x - first, blockIdx.z);
}

}  // namespace mavg
