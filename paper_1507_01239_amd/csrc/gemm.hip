// fp32 GEMM on the CDNA4 matrix cores with the fused epilogues the training path needs and a deterministic split of the
// contraction for problems with too few output tiles to fill 256 compute units.
//
// This file: the plan (kernel family, tile shape, splits), the dispatch to the kernel families, the split-contraction
// reducer and the exported entry points.  The kernels live in gemm_device.h and gemm_split.h and are instantiated per
// family in gemm_split*.hip, gemm_dma64.hip, gemm_kg.hip, gemm_kg64.hip and gemm_legacy.hip (separate files so that they compile in
// parallel).  They share the epilogues, the tile order and the split-contraction reducer:
//  - gemm_split_kernel: every fp32 element in two fp16 parts, three fp16 MFMAs (v_mfma_f32_32x32x16_f16) per product, or in
//    three bf16 parts, six bf16 MFMAs; tiles from 32x64 to 256x128, any alignment: everything large, and everything the next two
//    cannot take;
//  - gemm_dma_kernel (v_mfma_f32_32x32x2_f32), gemm_dma_kg_kernel and gemm_kg64_kernel (two fp16 parts, made when a wavefront reads its operands back,
//    or the same MFMA):
//    operands go from global memory straight into an LDS ring (global_load_lds_dwordx4): problems that do not fill the chip
//    with large tiles, 16-byte aligned rows;
//  - gemm_kernel: register-staged 64x64 tiles of the same MFMA with guarded loads, for what is left (contractions of fewer
//    than 32 steps, fused row sums of ragged operands).
#include "gemm_device.h"
#include "gemm_launchers.h"
#include "gemm_packed.h"
#include "packed.h"

namespace mavg {

// Sum the partial results of a split contraction in split order and apply the epilogue.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmKParams p) {
    const int b = blockIdx.y;
    const int64_t MN = (int64_t)p.M * p.N;
    const EpiCtx c = epi_ctx(p.epi, p.C, p.c_bstride, b);
    const float* __restrict__ W = p.ws + (int64_t)b * p.splits * MN;
    if ((p.N & 3) == 0) {
        const int64_t nq = MN >> 2;
        for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < nq; q += (int64_t)gridDim.x * 256) {
            // request all (at most 16) partial sums before adding any: one memory latency, not one per few splits
            float4 t[16];
#pragma unroll
            for (int sp = 0; sp < 16; ++sp)
                if (sp < p.splits) t[sp] = *reinterpret_cast<const float4*>(W + sp * MN + q * 4);
            float4 s = t[0];
#pragma unroll
            for (int sp = 1; sp < 16; ++sp)
                if (sp < p.splits) { s.x += t[sp].x; s.y += t[sp].y; s.z += t[sp].z; s.w += t[sp].w; }
            for (int sp = 16; sp < p.splits; ++sp) {
                const float4 u = *reinterpret_cast<const float4*>(W + sp * MN + q * 4);
                s.x += u.x; s.y += u.y; s.z += u.z; s.w += u.w;
            }
            const int64_t e = q * 4;
            const int m = (int)(e / p.N), n = (int)(e - (int64_t)m * p.N);
            MAVG_EPI_DISPATCH(p.epi.kind, (epi_apply4<KIND>(p.epi, c, p.ldc, p.N, m, n, s)))
        }
    } else {
        for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < MN; e += (int64_t)gridDim.x * 256) {
            float t[16];
#pragma unroll
            for (int sp = 0; sp < 16; ++sp)
                if (sp < p.splits) t[sp] = W[sp * MN + e];
            float s = t[0];
#pragma unroll
            for (int sp = 1; sp < 16; ++sp)
                if (sp < p.splits) s += t[sp];
            for (int sp = 16; sp < p.splits; ++sp) s += W[sp * MN + e];
            const int m = (int)(e / p.N), n = (int)(e - (int64_t)m * p.N);
            MAVG_EPI_DISPATCH(p.epi.kind, (epi_apply<KIND>(p.epi, c, p.ldc, p.N, m, n, s)))
        }
    }
}

// ---- host side -----------------------------------------------------------------------------------

struct TileCfg { int bm, bn, bk, threads; };
// indexed by GemmCfg
static const TileCfg kCfgs[CFG_COUNT] = {
    {64, 64, 16, 256},     // CFG_64
    {64, 64, 16, 256},     // CFG_64_REG
    {256, 128, 16, 512},   // CFG_S256
    {64, 64, 16, 256},     // CFG_S64
    {64, 128, 16, 512},    // CFG_S64x128
    {128, 128, 16, 512},   // CFG_S128
    {64, 64, 16, 256},     // CFG_64_RING3
    {32, 64, 16, 512},     // CFG_KG_32x64
    {32, 32, 16, 256},     // CFG_KG_32x32
    {32, 64, 16, 512},     // CFG_S32x64
    {64, 64, 16, 256},     // CFG_KG_64x64
    {64, 128, 16, 256},    // CFG_KG_64x128
};
constexpr int kNumCfgs = CFG_COUNT;
static inline bool cfg_kg(int cfg) { return cfg == CFG_KG_32x64 || cfg == CFG_KG_32x32 || cfg >= CFG_KG_64x64; }
static inline bool cfg_split(int cfg) { return (cfg >= CFG_S256 && cfg <= CFG_S128) || cfg == CFG_S32x64; }
static inline int64_t tiles_of(int cfg, int M, int N, int batch) {
    return (int64_t)((M + kCfgs[cfg].bm - 1) / kCfgs[cfg].bm) * ((N + kCfgs[cfg].bn - 1) / kCfgs[cfg].bn) * batch;
}

// The plan without the split-operand kernels (or the configuration that is asked for).
static GemmPlan gemm_plan_direct(int M, int N, int K, int batch, int force_cfg, int force_splits) {
    GemmPlan pl;
    // Measured on MI355X (layer shapes at minibatch 256 to 1024, 1 and 8 replicas): the 64x64 direct-to-LDS
    // kernel wins everywhere; many small workgroups per compute unit run out of phase and hide each other's
    // load, barrier and epilogue latencies.
    int cfg = force_cfg;
    // A short contraction over many tiles (the weight gradients: K is the minibatch) runs better with a ring of
    // three stages: a quarter less LDS lets one more workgroup share the compute unit, and it is the overlap of
    // one workgroup's read-modify-write epilogue with its neighbours' multiplies that is short there
    // (8000x2048x256: 90 against 95 us); the long contractions want the deeper ring (256x8000x2048: 73 against 81).
    if (cfg < 0 || cfg >= kNumCfgs) {
        const int64_t t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch;
        cfg = (K <= 1024 && t64 >= 1024) ? CFG_64_RING3 : CFG_64;
        // A skinny problem whose 32x64 tiles come to about one per compute unit (the 256 x 2048 x 2048 hidden
        // layers of the minibatch-256 step) does its contraction split inside the workgroup: with fp32 MFMAs in both
        // 21 to 23 against 26.9 us including the reducer (13.1 against 15.9 us for the 440-wide first layer).  Not at half or
        // twice that many tiles, nor for K = 8000 (measured).  (With fp16 parts it is a candidate of gemm_plan by its cost.)
        const int64_t t3264 = (int64_t)((M + 31) / 32) * ((N + 63) / 64) * batch;
        // (One workgroup of it fills a compute unit's LDS: past one tile per compute unit the launch takes two turns, with fp32
        // MFMAs 39 us at 272 or 288 rows against 29 us for 64x64 tiles split in three.)
        if (cfg == CFG_64 && t3264 >= 3 * kNumCU / 4 && t3264 <= kNumCU && K >= 256 && K <= 4096) cfg = CFG_KG_32x64;
        // Half as many rows again (128 x 2048 x 2048): 32x32 tiles, one wavefront per k-group, no barrier in the
        // loop, with fp32 MFMAs: 18.0 against 19.8 us.  (Two of its workgroups share a compute unit.)
        const int64_t t3232 = (int64_t)((M + 31) / 32) * ((N + 31) / 32) * batch;
        if (cfg == CFG_64 && t3232 >= 3 * kNumCU / 4 && t3232 <= kNumCU + kNumCU / 8 && K >= 1024 && K <= 4096) cfg = CFG_KG_32x32;
    }
    pl.cfg = cfg;
    pl.bm = kCfgs[cfg].bm; pl.bn = kCfgs[cfg].bn;
    const int bk = kCfgs[cfg].bk;
    const int64_t tiles = (int64_t)((M + pl.bm - 1) / pl.bm) * ((N + pl.bn - 1) / pl.bn) * batch;
    int splits = cfg_kg(cfg) ? (cfg == CFG_KG_64x128 && force_splits > 1 ? force_splits : 1) : force_splits;      // the others split the contraction inside the workgroup only
    if (splits <= 0) {
        // A launch takes about as long as the workgroups of its fullest compute unit one after the other: in units of
        // contraction steps, ceil(tiles * splits / compute units) * K / splits; a compute unit with a single, short
        // workgroup (fewer than 6000 steps) has nothing to hide its prologue and epilogue behind (+ 20 %); the reducer
        // costs 6 us (340 steps' worth at 64x64) and each split 8 bytes per element of C at about 4 TB/s.  Splits keep at
        // least 16 k-tiles each, and a split must promise 5 % to be taken.  Measured with 64x64 tiles (us for the
        // splits named, the model's choice marked):
        //   28 tiles, K 2048:  6 / 8* / 10 / 16: 13.9 / 13.2 / 15.3 / 15.0       32 tiles, K 8000: 4 / 8* / 16: 37.5 / 25.8 / 27.6
        //   96 tiles, K 8000:  2 / 3 / 4 / 5*: 68 / 84 / 66 / 58                 128 tiles, K 8000: 2 / 3 / 4* / 5: 81 / 86 / 72 / 79
        //   160 tiles, K 2048: 1 / 2 / 3* / 4: 36 / 38 / 29 / 32                 192 tiles, K 2048: 1 / 2 / 3 / 4*: 36 - 39 / 38 / 39 / 34
        //   224, 256 tiles, K 2048: 1* / 2: 36 / 38.5, 37 / 40                   256 tiles, K 8000: 1* / 2 / 4: 127 / 129 / 132
        //   320 tiles, K 2048: 1 / 2: 63.5 / 55.9 (3* by the model)              384 tiles, K 2048: 1 / 2* / 3: 63.6 / 58.5 / 70.8
        //   384 tiles, K 8000: 1 / 2*: 231 / 193                                 512 tiles, K 2048: 1* / 2: 67 / 75
        //   500 and 625 tiles, K 2048: unsplit faster than split in two (no split is considered from 512 tiles on)
        splits = 1;
        if (tiles < 2 * kNumCU) {
            const int ktiles = (K + bk - 1) / bk;
            const double per_split = (double)M * N * batch * 1.14e-4;
            auto cost = [&](int sp) {
                const int64_t rounds = (tiles * sp + kNumCU - 1) / kNumCU;
                const int steps = (ktiles + sp - 1) / sp * bk;
                double c = (double)rounds * steps;
                if (rounds == 1 && steps < 6000) c *= 1.2;
                if (sp > 1) c += 340.0 + sp * per_split;
                return c;
            };
            int smax = K / (16 * bk);
            if (smax > 16) smax = 16;
            double best = cost(1);
            for (int sp = 2; sp <= smax; ++sp) {
                const double c = cost(sp);
                if (c < 0.95 * best) { best = c; splits = sp; }
            }
        }
    }
    // contraction elements per split, rounded up to the k tile; drop empty trailing splits
    int kper = ((K + splits - 1) / splits + bk - 1) / bk * bk;
    if (kper < bk) kper = bk;
    splits = (K + kper - 1) / kper;
    if (splits < 1) splits = 1;
    pl.splits = splits;
    return pl;
}

// Estimated microseconds of a launch (and its reducer): a launch ends with its fullest compute unit, which works through
// `rounds` workgroups of ks contraction steps each; the more compute units are busy, the longer each of them takes (power, L2).
//   c0 + rounds (c1 + c2 ks) + (rounds == 1: c3 ks) + workgroups / 256 (c4 + c5 ks),   reducer: c6 + c7 per MB of partial sums
// Coefficients: least squares of relative errors over 1500 shapes of 16 - 8192 x 32 - 9000 x 32 - 9000, each timed with every
// configuration and 1, 2, 4 and 8 splits in a captured graph (operands of ordinary values; standard deviations 5 - 8 %, 10 % for
// the register-staged kernel).
static double plan_cost(const GemmPlan& pl, int M, int N, int K, int batch, bool ragged) {
    struct Fit { double c0, c1, c2, c3, c4, c5, c6, c7; };
    static const Fit kDma64 = {2.97, 0.51, 0.01363, 0.00111, 0.56, 0.00201, 2.56, 0.156}, kReg64 = {3.43, 0, 0.02797, 0.01245, 0.31, 0.00737, 2.87, 0.464},
                     kKg32x64 = {2.08, 2.37, 0.00383, 0, 0, 0.00372, 0, 0}, kKg32x32 = {3.10, 0.60, 0.00316, 0.00133, 0, 0.00123, 0, 0},
                     kS256 = {3.85, 4.32, 0.03265, 0.00035, 4.07, 0.01120, 1.98, 0.163}, kS128 = {3.16, 7.53, 0.01804, 0.00007, 1.99, 0.00795, 2.91, 0.171},
                     kS64x128 = {3.12, 6.94, 0.01251, 0, 1.78, 0.00515, 2.71, 0.156}, kS64 = {4.37, 1.79, 0.00736, 0.00481, 0.38, 0.00435, 2.95, 0.101},
                     kS32x64 = {2.17, 5.02, 0.00461, 0.00001, 0.47, 0.00332, 2.86, 0.054};
    const Fit& f = pl.cfg == CFG_S256 ? kS256 : pl.cfg == CFG_S128 ? kS128 : pl.cfg == CFG_S64x128 ? kS64x128 : pl.cfg == CFG_S64 ? kS64
                 : pl.cfg == CFG_S32x64 ? kS32x64 : pl.cfg == CFG_KG_32x64 ? kKg32x64 : pl.cfg == CFG_KG_32x32 ? kKg32x32 : ragged ? kReg64 : kDma64;
    const int64_t w = tiles_of(pl.cfg, M, N, batch) * pl.splits;
    const double rounds = (double)((w + kNumCU - 1) / kNumCU), share = (double)w / kNumCU, ks = (double)K / pl.splits;
    double c = f.c0 + rounds * (f.c1 + f.c2 * ks) + share * (f.c4 + f.c5 * ks);
    if (rounds == 1) c += f.c3 * ks;
    if (pl.splits > 1) c += f.c6 + f.c7 * (8e-6 * pl.splits * M * N * batch);
    return c;
}

// The same with three parts (and fp32 MFMAs in the in-workgroup-split kernels), from measurements at 32 to 4096 rows, 440 to 8000
// contraction steps and 1 to 2000 tiles (operands of ordinary values: with every compute unit busy the split-operand kernels run
// into the power limit, which the share `full` of busy compute units stands for; on zeros they take a quarter less).
static double plan_cost_three(const GemmPlan& pl, int M, int N, int K, int batch, bool ragged) {
    const int64_t w = tiles_of(pl.cfg, M, N, batch) * pl.splits;
    const double rounds = (double)((w + kNumCU - 1) / kNumCU), full = w < kNumCU ? (double)w / kNumCU : 1.0;
    const double ks = (double)((K + pl.splits - 1) / pl.splits);
    double c;
    switch (pl.cfg) {
    case CFG_S128: c = 3 + rounds * (9 + ks * (0.0284 + 0.0131 * full * full)); break;
    case CFG_S64x128: c = 3 + rounds * (5 + ks * (0.0180 + 0.0055 * full * full)); break;
    case CFG_S64: c = 5 + rounds * (2 + ks * 0.0132) + (rounds == 1 ? ks * 0.005 : 0.0); break;      // (up to three workgroups per compute unit)
    case CFG_S32x64: c = 2.3 + rounds * (5.7 + ks * 0.0077); break;
    case CFG_KG_32x64: c = 5 + rounds * ks * 0.0075; break;
    case CFG_KG_32x32: c = 5 + (w < kNumCU ? 1.0 : (double)w / kNumCU) * ks * 0.0049; break;      // (two workgroups per compute unit)
    default:      // (64x64 tiles; measured at 1200 shapes: within 6 % of this, one standard deviation)
        if (ragged) c = 5 + rounds * ks * 0.0348 * (rounds == 1 ? 1.2 : 1.0);
        else c = pl.splits > 1 ? 3 + rounds * ks * 0.0145 : 5 + rounds * ks * 0.0157;
        break;
    }
    if (pl.splits > 1) {
        // the reducer and the partial sums; next to the split-operand kernels less of it shows, as their own epilogue is then
        // a plain store
        const double bytes = 8.0 * pl.splits * M * N * batch;
        c += cfg_split(pl.cfg) ? 3.5 + bytes / 20e6 + (bytes > 32e6 ? (bytes - 32e6) / 8e6 : 0.0) : 4 + bytes / 6e6;
    }
    return c;
}

// The automatic plans take the split-operand kernels from this many contraction steps on: where they sum shorter ones their
// errors are larger than those of the fp32 MFMAs.  Relative errors against float64, split / fp32, of terms of either sign and
// of positive terms: 16 steps 89 / 73 and 45 / 62 (e-9), 24 steps 93 / 89 and 43 / 74, 32 steps 94 / 103 and 45 / 84.
// The grouped launch's weight updates: from 80 steps on (99 / 161 and 46 / 138), below it they are memory's business anyway.
constexpr int kSplitMinK = 32, kSplitGroupedMinK = 80;

// Which kernel family: the cheapest by plan_cost among the plan without the split-operand kernels, the in-workgroup-split and the split-operand
// kernels, unsplit or with 2, 4 or 8 contraction splits of at least 256 steps.  Over the 1500 shapes the choice is 0.6 % above the
// fastest that was measured, and 12 % below the plans made for three bf16 parts (more than 10 % above those in twenty, short
// or small ragged products).  Measured (us; those plans against these):
//   4096 x 4096 x 4096: 686 / 405 (256x128)            8192 x 2048 x 2048: 349 / 210 (256x128)       2048 x 16384 x 512: 194 / 131 (256x128)
//   1999 x 8000 x 2048: 345 / 207 (256x128)            1999 x 2048 x 2048: 91 / 63 (128x128)         1024 x 2048 x 2048: 54 / 40 (64x128)
//   256 x 8000 x 2048: 54 / 43 (256x128, 4 splits; 64x128 42)                256 x 2048 x 8000: 56 / 45 (128x128, 8 splits)    200 x 3003 x 1021: 28 / 19 (64x64)
//   377 x 408 x 328: 9.3 / 5.7 (32x32 in-workgroup split)     22 x 7688 x 320: 8.3 / 5.4 (likewise)      256 x 2048 x 2048: 21 / 16 (32x64 likewise)
// (Two parts.  With three, small products stay with the fp32 MFMAs: every operand element has to be split once per tile it is used
// in, and LDS takes the parts at 64 bytes per cycle, which small tiles cannot hide.)
GemmPlan gemm_plan(int M, int N, int K, int batch, int force_cfg, int force_splits, bool ragged, int64_t ws_floats, bool three) {
    GemmPlan best = gemm_plan_direct(M, N, K, batch, force_cfg, force_splits);
    if ((force_cfg >= 0 && force_cfg < kNumCfgs) || K < kSplitMinK) return best;
    if (ragged && best.cfg != CFG_64) best = gemm_plan_direct(M, N, K, batch, CFG_64_REG, force_splits);
    auto cost = [&](const GemmPlan& pl) { return three ? plan_cost_three(pl, M, N, K, batch, ragged) : plan_cost(pl, M, N, K, batch, ragged); };
    // (what another kernel must promise: the estimates' scatter)
    double least = (three ? ragged ? 0.9 : 0.97 : 0.94) * cost(best);
    // Summation error: three parts have at least 0.75 times as many partial sums as the plan they replace.
    const int sums = three ? best.splits * (cfg_kg(best.cfg) ? 4 : 1) : 0;
    auto consider = [&](int cfg, int sp) {
        const GemmPlan pl = gemm_plan_direct(M, N, K, batch, cfg, sp);
        const double c = cost(pl);
        if (c < least) { least = c; best = pl; }
    };
    // (a k-tile of 16 steps for each of their wavefronts)
    if (!ragged && !three && force_splits <= 1) {
        if (K >= 16 * 8) consider(CFG_KG_32x64, 1);
        if (K >= 16 * 4) consider(CFG_KG_32x32, 1);
    }
    static const struct { int cfg, kgroups; } kSplitCfgs[] = {{CFG_S256, 1}, {CFG_S128, 2}, {CFG_S64x128, 4}, {CFG_S64, 2}, {CFG_S32x64, 8}};
    for (const auto& sc : kSplitCfgs)
        for (int sp = 1; sp <= 8; sp *= 2) {
            if (force_splits > 0 && sp != force_splits) continue;
            if (sp > 1 && (K < 256 * sp || (int64_t)sp * batch * M * N > ws_floats)) continue;
            if ((three && sc.cfg == CFG_S256) || 4 * sp * sc.kgroups < 3 * sums) continue;
            consider(sc.cfg, sp);
        }
    return best;
}

static int64_t plan_floats(const GemmPlan& pl, int M, int N, int batch) { return pl.splits > 1 ? (int64_t)pl.splits * batch * M * N : 0; }

// The plans without the split-operand kernels for one problem: the automatic one, and the register-staged one that takes its place where operands
// are not 16-byte aligned or their strides are too long for the others (an in-workgroup-split plan has no partial sums, the
// register-staged one for the same sizes up to sixteen splits of them).
static int64_t plan_floats_direct(int M, int N, int K, int batch, int cfg, int force_splits) {
    const int64_t f = plan_floats(gemm_plan_direct(M, N, K, batch, cfg, force_splits), M, N, batch);
    const int64_t g = plan_floats(gemm_plan_direct(M, N, K, batch, CFG_64_REG, force_splits), M, N, batch);
    return f > g ? f : g;
}

int64_t gemm_ws_floats_direct(int M, int N, int K, int batch) { return plan_floats_direct(M, N, K, batch, CFG_AUTO, 0); }

int64_t gemm_ws_floats(int M, int N, int K, int batch, int force_cfg, int force_splits) {
    const bool forced = force_cfg >= 0 && force_cfg < kNumCfgs;
    int64_t f = plan_floats_direct(M, N, K, batch, forced ? CFG_64_REG : CFG_AUTO, force_splits);
    // (Below 512 steps the split-operand kernels run unsplit when they are chosen, so those plans are all there is to
    // cover; callers ask on every call, and the comparison of plans is most of the host time of a small one.)
    if (!forced && force_splits <= 0 && K < 512) return f;
    auto cover = [&](const GemmPlan& pl) { const int64_t g = plan_floats(pl, M, N, batch); if (g > f) f = g; };
    cover(gemm_plan(M, N, K, batch, force_cfg, force_splits));
    cover(gemm_plan(M, N, K, batch, force_cfg, force_splits, true));
    return f;
}

static bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

// May the direct-to-LDS kernel run this problem?  Its loads are unmasked 16-byte loads.
static bool dma_eligible(const GemmDesc& d, const GemmKParams& p) {
    if (!p.vecA || !p.vecB) return false;
    if (d.K < kDmaBK || p.kper % kDmaBK != 0) return false;      // (a contraction tail of fewer than 16 steps is handled)
    if (!d.a_kc && (p.Mr < 4 || p.Mr % 4 != 0 || p.Mr > d.lda)) return false;
    if (!d.b_kc && (p.Nr < 4 || p.Nr % 4 != 0 || p.Nr > d.ldb)) return false;
    const int64_t lim = (int64_t)1 << 29;      // per-lane offsets are 32-bit byte offsets
    if ((d.a_kc ? (int64_t)d.M * d.lda : kDmaBK * d.lda + d.M) >= lim) return false;
    if ((d.b_kc ? (int64_t)d.N * d.ldb : kDmaBK * d.ldb + d.N) >= lim) return false;
    return true;
}

// May the split-operand kernels run this problem?  Their per-lane offsets inside a tile are 32-bit byte offsets, and their
// loads of whole k-tiles need 16 contraction steps.
static bool split_eligible(const GemmDesc& d) {
    const int64_t lim = (int64_t)1 << 22;
    return d.K >= 16 && d.lda < lim && d.ldb < lim;
}

static GemmKParams fill_params(const GemmDesc& d, const GemmPlan& pl, float* ws) {
    GemmKParams p;
    p.A = d.A; p.lda = d.lda; p.a_bstride = d.a_bstride;
    p.B = d.B; p.ldb = d.ldb; p.b_bstride = d.b_bstride;
    p.C = d.C; p.ldc = d.ldc; p.c_bstride = d.c_bstride;
    p.M = d.M; p.N = d.N; p.K = d.K; p.batch = d.batch;
    p.Mr = d.a_pad4 ? (d.M + 3) / 4 * 4 : d.M;
    p.Nr = d.b_pad4 ? (d.N + 3) / 4 * 4 : d.N;
    p.splits = pl.splits;
    const int bk = kCfgs[pl.cfg].bk;
    int kper = ((d.K + pl.splits - 1) / pl.splits + bk - 1) / bk * bk;
    if (kper < bk) kper = bk;
    p.kper = kper;
    p.tiles_m = (d.M + pl.bm - 1) / pl.bm;
    p.tiles_n = (d.N + pl.bn - 1) / pl.bn;
    p.vecA = aligned16(d.A) && (d.lda % 4 == 0) && (d.a_bstride % 4 == 0);
    p.vecB = aligned16(d.B) && (d.ldb % 4 == 0) && (d.b_bstride % 4 == 0);
    p.ws = ws;
    p.scale_a = ldexpf(1.f, d.a_exp); p.scale_b = ldexpf(1.f, d.b_exp);
    p.least_a = d.a_exact ? 0.f : kSplitLeast;
    p.three = d.parts == kThreeParts;
    p.epi = d.epi;
    return p;
}

// Short contractions in small tiles are split into three parts all the same: what two parts, or the look at the operands, cost once per
// tile is more than what they save.  Rows that are not 16-byte aligned, us in a captured graph, three parts / two / by data:
//   145 x 145: 129 steps 7.9 / 8.4 / 8.8, 193 steps 8.7 / 8.7 / 9.5, 385 steps 10.0 / 9.3 / 10.0      501 x 1501: 129 steps 9.4 / 8.9 / 9.3
static bool short_three(const GemmDesc& d, bool ragged) {
    return ragged && d.K < (d.parts == kPartsByData ? 384 : 192) && tiles_of(CFG_S32x64, d.M, d.N, d.batch) <= kNumCU;
}

// 64x64 or 64x128 tiles split four ways inside the workgroup, where that leaves few compute units idle and asks none to take a second turn (one
// of its workgroups fills a compute unit's LDS), for contractions in which the in-workgroup sum's few microseconds don't count while the
// partial sums and the reducer of a split across workgroups do, or the rounds and fixed costs of the split-operand kernels.  Two fp16 parts, time
// with / without over 200 shapes of 64 to 2900 rows, B from the last-level cache or from HBM:
// 64x64, 131 - 256 tiles, 512 - 2304 steps: 0.68 - 0.97, two shapes 1.00 (512x2048x2048 24.0 / 33.0 us, n-contiguous B 25.1 / 33.8, from HBM
//   30.0 / 33.7, 29.0 / 34.0; 384x2048x2048 22.2 / 29.8; 1769x296x1264 15.8 / 21.0); where 32x64 tiles need one turn 1.26 - 1.41;
//   280 - 464 steps 1.03 - 1.2; 2400 - 4224 steps 0.74 - 1.14, 4300 and more 0.88 - 1.4; 100 - 126 tiles 1.2 - 1.4; 316 and more 1.03 - 1.9
// 64x128 (where the 64x64 tiles are too many), 192 - 256 tiles, 512 - 2304 steps, rows that begin at 64-byte boundaries: 0.79 - 0.97, one shape 1.02
//   (1024x2048x2048 41.8 / 48.1 us, n-contiguous B 38.6 / 48.1, from HBM 43.5 / 49.6, 39.2 / 49.5; 768x2048x2048 34.2 / 40.0); other
//   rows, whose 64-byte pieces lie in two cache lines, up to 1.07; 130 - 188 tiles 0.80 - 1.28; 320 - 500 steps 0.9 - 1.14; 2400 and more
//   0.9 - 1.17; 270 tiles and more 1.04 - 1.4
// 64x128 and n-contiguous B (a back-propagated error by its weights), contractions of more than 2304 steps, from HBM, over 60 shapes:
//   unsplit 0.75 - 0.95 (1024x2048x8000 117 / 124 us); two splits across workgroups of 1240 - 2048 steps each 0.80 - 0.93 (192x4480x2880 38 / 45), longer ones
//   0.75 - 1.04; four of 1200 steps and more 0.82 - 0.97 (256x2048x8000 47 / 51), shorter ones 0.88 - 1.28.  (k-contiguous B: 0.9 - 1.17)
// Returns the configuration, CFG_AUTO for none, and the splits.
static int kg64_plan(const GemmDesc& d, int64_t ws_floats, int& splits) {
    splits = 1;
    if (d.force_cfg >= 0 || d.force_splits > 1 || d.K < 512 || d.K > 9000) return CFG_AUTO;
    const int64_t t64 = tiles_of(CFG_KG_64x64, d.M, d.N, d.batch), t128 = tiles_of(CFG_KG_64x128, d.M, d.N, d.batch);
    auto full_round = [&](int sp) { return 4 * t128 * sp >= 3 * kNumCU && t128 * sp <= kNumCU; };
    auto starts_at_64 = [](const float* q, int64_t ld, int64_t stride) { return ((reinterpret_cast<uintptr_t>(q) | (uintptr_t)ld * 4 | (uintptr_t)stride * 4) & 63) == 0; };
    const bool lines = starts_at_64(d.A, d.lda, d.a_bstride) && starts_at_64(d.B, d.ldb, d.b_bstride);
    if (d.K > 2304) {
        if (d.b_kc || !lines) return CFG_AUTO;
        if (full_round(1)) return CFG_KG_64x128;
        if (full_round(2) && d.K >= 2 * 1240 && d.K <= 2 * 2048) splits = 2;
        else if (full_round(4) && d.K >= 4 * 1200) splits = 4;
        return splits > 1 && d.force_splits == 0 && (int64_t)splits * d.batch * d.M * d.N <= ws_floats ? CFG_KG_64x128 : CFG_AUTO;
    }
    if (t64 <= kNumCU) return 2 * t64 > kNumCU && tiles_of(CFG_KG_32x64, d.M, d.N, d.batch) > kNumCU ? CFG_KG_64x64 : CFG_AUTO;
    return full_round(1) && lines ? CFG_KG_64x128 : CFG_AUTO;
}

int gemm_launch(const GemmDesc& d, float* ws, int64_t ws_floats, hipStream_t stream) {
    if (d.M <= 0 || d.N <= 0 || d.batch <= 0) return 0;
    if (d.epi.rowsum_dst != nullptr && d.a_kc) return note_hip_error(hipErrorInvalidValue);
    // fused row sums and the side sum are the work of the kernels that own a whole tile: unsplit, no k-groups
    const bool rowsum = d.epi.rowsum_dst != nullptr || d.epi.side_sum_src != nullptr;
    GemmPlan pl = gemm_plan_direct(d.M, d.N, d.K, d.batch, rowsum && cfg_split(d.force_cfg) ? CFG_64 : d.force_cfg, rowsum ? 1 : d.force_splits);
    GemmKParams p = fill_params(d, pl, ws);
    bool three = d.parts == kThreeParts;
    if (!rowsum && split_eligible(d)) {
        const bool ragged = !dma_eligible(d, p);
        three = three || (d.force_cfg < 0 && short_three(d, ragged));
        int kg64_splits = 1;
        const int kg64 = three || ragged ? CFG_AUTO : kg64_plan(d, ws ? ws_floats : 0, kg64_splits);
        pl = kg64 != CFG_AUTO ? gemm_plan_direct(d.M, d.N, d.K, d.batch, kg64, kg64_splits)
                              : gemm_plan(d.M, d.N, d.K, d.batch, d.force_cfg, d.force_splits, ragged, ws ? ws_floats : 0, three);
        p = fill_params(d, pl, ws);
    }
    if ((cfg_split(pl.cfg) && !split_eligible(d)) ||
        (cfg_kg(pl.cfg) && !(dma_eligible(d, p) && !rowsum && d.K / kDmaBK >= (pl.cfg == CFG_KG_32x64 ? 2 : 1) * kKGroups))) {
        pl = gemm_plan_direct(d.M, d.N, d.K, d.batch, CFG_64_REG, rowsum ? 1 : d.force_splits);
        p = fill_params(d, pl, ws);
    }
    if (pl.splits > 1 && (ws == nullptr || ws_floats < (int64_t)pl.splits * d.batch * d.M * d.N)) return note_hip_error(hipErrorInvalidValue);
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), 1, (unsigned)(d.batch * pl.splits));
    if (cfg_split(pl.cfg)) {      // (the plan may have been replaced above)
        typedef void (*Launch)(const GemmKParams&, bool, bool, dim3, hipStream_t);
        static const Launch k256[] = {launch_split256_three, launch_split256, launch_split256_by_data},
                            k128[] = {launch_split128_three, launch_split128, launch_split128_by_data},
                            k64x128[] = {launch_split64x128_three, launch_split64x128, launch_split64x128_by_data},
                            k64[] = {launch_split64_three, launch_split64, launch_split64_by_data},
                            k32x64[] = {launch_split32x64_three, launch_split32x64, launch_split32x64_by_data};      // (in the order of SplitParts)
        const Launch* of = pl.cfg == CFG_S256 ? k256 : pl.cfg == CFG_S64x128 ? k64x128 : pl.cfg == CFG_S64 ? k64 : pl.cfg == CFG_S32x64 ? k32x64 : k128;
        of[three ? kThreeParts : d.parts](p, d.a_kc, d.b_kc, grid, stream);
    } else if (pl.cfg >= CFG_KG_64x64) launch_kg64(pl.cfg, p, d.a_kc, d.b_kc, grid, stream);
    else if (cfg_kg(pl.cfg)) launch_kg(pl.cfg, p, d.a_kc, d.b_kc, grid, stream);
    else if (pl.cfg != CFG_64_REG && dma_eligible(d, p)) launch_dma64(pl.cfg, p, d.a_kc, d.b_kc, grid, stream);
    else launch_legacy(p, d.a_kc, d.b_kc, grid, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return note_hip_error(e);
    if (pl.splits > 1) {
        // one float4 per thread when rows are multiples of 4 long, else one element per thread
        const int64_t work = (d.N & 3) == 0 ? (int64_t)d.M * d.N / 4 : (int64_t)d.M * d.N;
        int64_t gx = (work + 255) / 256;
        if (gx > 4096) gx = 4096;
        if (gx < 1) gx = 1;
        hipLaunchKernelGGL(gemm_reduce_kernel, dim3((unsigned)gx, (unsigned)d.batch), dim3(256), 0, stream, p);
        e = hipGetLastError();
    }
    return note_hip_error(e);
}

// Thin products X R^T in one launch (see gemm_thin_grouped_kernel); a problem that kernel cannot take is launched by
// itself, unsplit.
static int gemm_launch_grouped_thin(const GemmDesc* d, int count, hipStream_t stream) {
    ThinGroupParams gp;
    gp.ngroups = 0;
    int tiles = 0, batch = 0;
    auto flush = [&]() -> int {
        if (gp.ngroups == 0) return 0;
        gp.tile_start[gp.ngroups] = tiles;
        launch_thin(gp, dim3((unsigned)tiles, 1, (unsigned)batch), stream);
        gp.ngroups = 0;
        tiles = 0;
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? 0 : note_hip_error(e);
    };
    for (int i = 0; i < count; ++i) {
        const GemmDesc& di = d[i];
        if (di.M <= 0 || di.N <= 0 || di.batch <= 0) continue;
        if (!di.a_kc || !di.b_kc || di.batch != d[0].batch || di.epi.kind != EPI_STORE || di.epi.rowsum_dst != nullptr)
            return note_hip_error(hipErrorInvalidValue);
        const GemmPlan pl = gemm_plan_direct(di.M, di.N, di.K, di.batch, CFG_KG_32x32, 1);
        const GemmKParams q = fill_params(di, pl, nullptr);
        if (!dma_eligible(di, q) || di.K / kDmaBK < kThinKGroups) {
            GemmDesc one = di;
            one.force_cfg = -1; one.force_splits = 1;
            if (gemm_launch(one, nullptr, 0, stream) != 0) return -1;
            continue;
        }
        batch = di.batch;
        ThinProblem& t = gp.g[gp.ngroups];
        t.A = di.A; t.B = di.B; t.C = di.C;
        t.lda = di.lda; t.ldb = di.ldb; t.ldc = di.ldc;
        t.a_bstride = di.a_bstride; t.b_bstride = di.b_bstride; t.c_bstride = di.c_bstride;
        t.M = di.M; t.N = di.N; t.K = di.K;
        gp.tile_start[gp.ngroups] = tiles;
        tiles += q.tiles_m * q.tiles_n;
        if (++gp.ngroups == kMaxThin && flush() != 0) return -1;
    }
    return flush();
}

static int64_t grouped_tiles128(const GemmDesc* d, int count) {
    int64_t t = 0;
    for (int i = 0; i < count; ++i) t += tiles_of(CFG_S128, d[i].M > 0 ? d[i].M : 0, d[i].N > 0 ? d[i].N : 0, d[i].batch);
    return t;
}

// Which kernel of the grouped launch takes problem d (q: its parameters for 64x64 tiles) among problems of tiles128 tiles in
// all: 0 = split-operand (128x128 tiles; m- and n-contiguous operands), 1 = direct-to-LDS, 2 = register-staged.
// The split-operand kernel takes it when the tiles come to at least four per compute unit, two from 512 steps on (with
// fewer the read-modify-write of C has nothing to hide behind: 140 tiles, two replicas of 1696 x 528 and 64 x 1696 at 270 rows,
// made the step 88 us, 73 with 64x64 tiles of fp32 MFMAs), and the contraction is long enough for its faster multiplies to
// matter next to that: the seven weight updates of 440-6x2048-8000 take 116 us on fp32 MFMAs at minibatch 128 (split-operand 140:
// backward passes of 8 replicas 1311 against 1344 us, at 64 rows 960 against 1134), 177 against 144 at 256, 318 against 202 at 512,
// 616 against 338 at 1024.
// Rows that are not 16-byte aligned: from half a tile per compute unit and kSplitGroupedMinK steps on (the alternative there
// is the register-staged kernel, 28 against 21 us at 3003 x 1021 x 200).
static int grouped_kernel(const GemmDesc& d, const GemmKParams& q, int64_t tiles128) {
    const bool dma = dma_eligible(d, q);
    const bool split = split_eligible(d) && !d.a_kc && !d.b_kc && d.epi.side_sum_src == nullptr &&
                       tiles128 >= (!dma ? kNumCU / 2 : d.K >= 512 ? 2 * kNumCU : 4 * kNumCU) && d.K >= (dma ? 192 : kSplitGroupedMinK);
    return split ? 0 : dma ? 1 : 2;
}

// Which tiles the split-operand kernel takes such a problem in: 256x128 where the contraction is long and the tiles are many (one
// workgroup per compute unit, whose epilogue nothing hides, but a third fewer elements to split per MFMA).  Backward passes of
// 440-6x2048-8000, us, 128x128 / 256x128 tiles:   512 rows: 1 replica 503 / 513, 2 846 / 880, 4 1493 / 1536, 8 2760 / 2834
//                                                1024 rows: 1 replica 777 / 780, 2 1347 / 1355, 4 2481 / 2461, 8 4972 / 4912
// (2352 tiles of 128x128 a replica: the line lies between two replicas and four)
static bool grouped_wide(const GemmDesc& d, int64_t tiles128) { return d.K >= 1024 && tiles128 >= 32 * kNumCU; }

int gemm_grouped_kernel(const GemmDesc* d, int count, int which) {
    return grouped_kernel(d[which], fill_params(d[which], gemm_plan_direct(d[which].M, d[which].N, d[which].K, d[which].batch, CFG_64, 1), nullptr),
                          grouped_tiles128(d, count));
}

int gemm_launch_grouped(const GemmDesc* d, int count, hipStream_t stream, bool thin) {
    if (thin) return gemm_launch_grouped_thin(d, count, stream);
    // Four passes over the problems, one for each kernel: split-operand (0 with 128x128 tiles, 3 with 256x128), 1 and 2.
    const int64_t tiles128 = grouped_tiles128(d, count);
    const bool three = count > 0 && d[0].parts == kThreeParts;
    for (int pass = 0; pass < 4; ++pass) {
        GemmGroupParams gp;
        gp.ngroups = 0;
        int tiles = 0, batch = 0;
        bool a_kc = false, b_kc = false;
        auto flush = [&]() -> int {
            if (gp.ngroups == 0) return 0;
            gp.tile_start[gp.ngroups] = tiles;
            const dim3 grid((unsigned)tiles, 1, (unsigned)batch);
            if (pass == 0 || pass == 3) (three ? launch_grouped_split_three : d[0].parts == kTwoParts ? launch_grouped_split : launch_grouped_split_by_data)(gp, pass == 3, grid, stream);
            else if (pass == 1) launch_grouped_dma(gp, a_kc, b_kc, grid, stream);
            else launch_grouped_legacy(gp, a_kc, b_kc, grid, stream);
            gp.ngroups = 0;
            tiles = 0;
            const hipError_t e = hipGetLastError();
            return e == hipSuccess ? 0 : note_hip_error(e);
        };
        for (int i = 0; i < count; ++i) {
            const GemmDesc& di = d[i];
            if (di.M <= 0 || di.N <= 0 || di.batch <= 0) continue;
            if (di.a_kc != d[0].a_kc || di.b_kc != d[0].b_kc || di.batch != d[0].batch) return note_hip_error(hipErrorInvalidValue);
            if (di.epi.rowsum_dst != nullptr && di.a_kc) return note_hip_error(hipErrorInvalidValue);
            if (di.parts != d[0].parts) return note_hip_error(hipErrorInvalidValue);
            // unsplit, 64x64 tiles (the split-operand kernel's below)
            GemmKParams q = fill_params(di, gemm_plan_direct(di.M, di.N, di.K, di.batch, CFG_64, 1), nullptr);
            const int kernel = grouped_kernel(di, q, tiles128);
            if ((kernel == 0 && !three && grouped_wide(di, tiles128) ? 3 : kernel) != pass) continue;
            if (kernel == 0) q = fill_params(di, gemm_plan_direct(di.M, di.N, di.K, di.batch, pass == 3 ? CFG_S256 : CFG_S128, 1), nullptr);
            a_kc = di.a_kc; b_kc = di.b_kc; batch = di.batch;
            gp.g[gp.ngroups] = q;
            gp.tile_start[gp.ngroups] = tiles;
            tiles += q.tiles_m * q.tiles_n;
            if (++gp.ngroups == kMaxGroups && flush() != 0) return -1;
        }
        if (flush() != 0) return -1;
    }
    return 0;
}

// ---- weight updates on packed operands ---------------------------------------------------------------

// Scratch of one operand, in floats: its packed form (an operand that the replicas share is packed once), its columns' exponents.
struct PackedOperand { int batch; int64_t floats, exps; };
static PackedOperand packed_operand(int rows, int cols, int batch, int64_t bstride, int pieces) {
    PackedOperand o;
    o.batch = batch > 1 && bstride == 0 ? 1 : batch;
    o.floats = ((int64_t)pieces * ((rows + 15) / 16) * 16 * cols + 63) / 64 * 64;
    o.exps = (cols + 255) / 256 * 256;
    return o;
}
constexpr int kPackWidthLeast = 16;      // columns per workgroup (see pack_kernel): partial sums of squares have room for that many
int64_t gemm_packed_floats(int M, int N, int K, int batch, int pieces) {
    const PackedOperand a = packed_operand(K, M, batch, 1, pieces), b = packed_operand(K, N, batch, 1, pieces);
    return batch * (a.floats + a.exps + b.floats + b.exps) + (pieces > 1 ? (N / kPackWidthLeast + 64) / 64 * 64 : 0);
}

// From kSplitGroupedMinK steps on, where fp16 parts sum no less exactly than fp32 MFMAs, and where the launch that packs (5 - 9 us, and some 3 us
// for the dependence between the two) is worth it: large updates, whose time is the parameters' way through memory, and the products of
// long contractions with a tile of 128x128 or more per compute unit.  A training step, us, without / with (rows, replicas):
//   440-6x2048-8000 (2352 tiles): 128 rows 368 / 337, 256 444 / 417           429-3x2047-8001 (1792 tiles): 128 rows 292 / 272
//   440-3x2048 (576): 256 134 / 133, 512 205 / 190       440-2048-2048 (320): 200 74.5 / 78.2, 512 120 / 117, 1024 203 / 180
//   440-3x1024-3000 (352): 200 124 / 127, 320 138 / 139, 512 180 / 168, 1024 295 / 265; 2 replicas (704) 256 183 / 186
//   440-3x1500 (336): 512 167 / 163, 1024 295 / 283      440-1024-1024, 4 replicas (384): 256 93.8 / 97.7, 512 150 / 145
//   440-3x512-4000 (176): 640 146 / 151, 1280 222 / 224
//   rows that are not 16-byte aligned: 429-3x1021-3003 (352) 200 167 / 172, 1000 309 / 312, 2000 471 / 463; 301-3x701-2005, 2 replicas (372) 512 230 / 240
// Of two pieces (statistics of an RBM) packing replaces the launch for the visible bias: 440 x 2048 with 2 x 256 rows 22 / 18.
bool gemm_packed_takes(const GemmDesc* d, int count, int pieces) {
    double flop = 0;
    int least = INT32_MAX;
    bool aligned = true;
    for (int i = 0; i < count; ++i) {
        if (d[i].a_kc || d[i].b_kc || d[i].epi.kind != EPI_AXPBY || !split_eligible(d[i])) return false;
        if (d[i].K * pieces < least) least = d[i].K * pieces;
        flop += 2.0 * d[i].M * d[i].N * d[i].K * pieces * d[i].batch;
        aligned = aligned && d[i].lda % 4 == 0 && d[i].ldb % 4 == 0;
    }
    if (count < 1 || least < kSplitGroupedMinK) return false;
    const int64_t tiles = grouped_tiles128(d, count);
    return tiles >= 4 * kNumCU || (pieces > 1 ? least >= 192 && flop >= 0.7e9 : aligned && least >= 448 && tiles >= kNumCU);
}

// Tiles: 64x64 below one tile of 128x128 per compute unit (440 x 2048 at 512 rows 11.4 us, 64x128 14.8), 128x128 for long contractions in
// many tiles (440-6x2048-8000: 512 rows 168 / 157 / 160, 768 270 / 204 / 197, 1000 366 / 252 / 240), 64x128 otherwise (three workgroups per
// compute unit hide each other's update: 128 rows 77 / 72 / 80, 256 107 / 90 / 98).
static int packed_shape(int K, int64_t tiles128) { return tiles128 < kNumCU ? 0 : K < 768 || tiles128 < 2 * kNumCU ? 1 : 2; }

int gemm_launch_packed(const GemmDesc* d, int count, float* ws, int64_t ws_floats, hipStream_t stream, int tiles, const PackedPieces* pieces) {
    const int npieces = pieces ? 2 : 1;
    int64_t need = 0;
    for (int i = 0; i < count; ++i) need += gemm_packed_floats(d[i].M, d[i].N, d[i].K, d[i].batch, npieces);
    if (ws_floats < need || (pieces && (count != 1 || d[0].batch != 1))) return note_hip_error(hipErrorInvalidValue);
    const int shape = tiles >= 0 ? tiles : packed_shape(d[0].K * npieces, grouped_tiles128(d, count));
    for (int i0 = 0; i0 < count; i0 += kMaxGroups) {
        PackedGroupParams gp;
        PackGroupParams pk;
        gp.ngroups = pk.ngroups = 0;
        int ntiles = 0, most_rows = 0;
        const int batch = d[i0].batch, end = count < i0 + kMaxGroups ? count : i0 + kMaxGroups;
        // columns per packing workgroup: whole cache lines where that leaves a workgroup per compute unit
        int64_t blocks64 = 0;
        for (int i = i0; i < end; ++i) blocks64 += ((int64_t)(d[i].M + 63) / 64 + (d[i].N + 63) / 64) * d[i].batch;
        const int width = blocks64 >= kNumCU ? 64 : blocks64 >= kNumCU / 2 ? 32 : kPackWidthLeast;
        int blocks = 0;
        for (int i = i0; i < end; ++i) {
            const GemmDesc& di = d[i];
            if (di.M <= 0 || di.N <= 0 || di.batch <= 0) continue;
            if (di.a_kc || di.b_kc || di.batch != batch || di.epi.kind != EPI_AXPBY) return note_hip_error(hipErrorInvalidValue);
            GemmPlan pl = gemm_plan_direct(di.M, di.N, di.K, di.batch, CFG_64, 1);
            pl.bm = kPackedTiles[shape].bm; pl.bn = kPackedTiles[shape].bn;
            PackedParams& q = gp.g[gp.ngroups];
            q.g = fill_params(di, pl, nullptr);
            q.kt = npieces * ((di.K + 15) / 16);
            q.A2 = pieces ? pieces->A2 : nullptr; q.B2 = pieces ? pieces->B2 : nullptr;
            q.lda2 = pieces ? pieces->lda2 : 0; q.ldb2 = pieces ? pieces->ldb2 : 0;
            auto pack = [&](const float* src, int64_t ld, int64_t bstride, int cols, const char*& packed, int64_t& pstride, const int32_t*& exps, int64_t& estride) -> PackMatrix& {
                const PackedOperand o = packed_operand(di.K, cols, di.batch, bstride, npieces);
                PackMatrix& m = pk.g[pk.ngroups];
                m = PackMatrix();
                m.src = src; m.ld = ld; m.bstride = bstride;
                m.dst = reinterpret_cast<char*>(ws); m.dst_bstride = o.floats * 4;
                m.exps = reinterpret_cast<int32_t*>(ws + o.batch * o.floats); m.e_bstride = o.exps;
                m.rows = di.K; m.cols = cols; m.batch = o.batch;
                packed = m.dst; exps = m.exps;
                pstride = o.batch == di.batch ? m.dst_bstride : 0; estride = o.batch == di.batch ? o.exps : 0;
                ws += o.batch * (o.floats + o.exps);
                pk.block_start[pk.ngroups++] = blocks;
                blocks += (cols + width - 1) / width;
                return m;
            };
            PackMatrix& ma = pack(di.A, di.lda, di.a_bstride, di.M, q.pa, q.pa_bstride, q.ea, q.e_bstride_a);
            const Epilogue& e = di.epi;
            if (e.rowsum_dst) {
                ma.sum_dst = e.rowsum_dst; ma.sum_bstride = e.rowsum_bstride; ma.sum_alpha = e.rowsum_alpha; ma.sum_beta = e.rowsum_beta;
                ma.sum_dst2 = e.rowsum_dst2; ma.sum2_bstride = e.rowsum2_bstride;
                ma.sum_w = e.rowsum_w; ma.sum_w_bstride = e.rowsum_w_bstride;
                ma.alpha_dev0 = e.alpha_dev0; ma.alpha_dev1 = e.alpha_dev1;
            }
            PackMatrix& mb = pack(di.B, di.ldb, di.b_bstride, di.N, q.pb, q.pb_bstride, q.eb, q.e_bstride_b);
            if (pieces) {
                ma.src2 = pieces->A2; ma.ld2 = pieces->lda2; ma.sum_sign2 = 1.f;
                mb.src2 = pieces->B2; mb.ld2 = pieces->ldb2; mb.sum_sign2 = -1.f;
                mb.sum_dst = pieces->diff_dst; mb.sum_alpha = pieces->diff_alpha; mb.sum_beta = pieces->diff_beta; mb.sum_dst2 = pieces->diff_dst2;
                if (pieces->square_dst) {
                    mb.sq_partial = ws;
                    q.g.epi.side_sum_src = ws; q.g.epi.side_sum_dst = pieces->square_dst; q.g.epi.side_sum_n = (di.N + width - 1) / width;
                }
            }
            gp.tile_start[gp.ngroups++] = ntiles;
            ntiles += q.g.tiles_m * q.g.tiles_n;
            if (di.K > most_rows) most_rows = di.K;
        }
        if (gp.ngroups == 0) continue;
        gp.tile_start[gp.ngroups] = ntiles;
        pk.block_start[pk.ngroups] = blocks;
        launch_pack(pk, width, npieces, most_rows, dim3((unsigned)blocks, (unsigned)batch), stream);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return note_hip_error(e);
        launch_grouped_packed(gp, shape, dim3((unsigned)ntiles, 1, (unsigned)batch), stream);
        e = hipGetLastError();
        if (e != hipSuccess) return note_hip_error(e);
    }
    return 0;
}

}  // namespace mavg

static thread_local hipError_t g_last_error = hipSuccess;
namespace mavg {
int note_hip_error(hipError_t e) {
    if (e != hipSuccess) g_last_error = e;
    return (int)e;
}
}  // namespace mavg

extern "C" const char* mavg_last_error(void) { return hipGetErrorString(g_last_error); }

// ---- exported test/tuning entry points -----------------------------------------------------------
using namespace mavg;

extern "C" int64_t mavg_gemm_workspace_bytes(int32_t m, int32_t n, int32_t k, int32_t cfg, int32_t splits) {
    if (m < 1 || n < 1 || k < 0) return MAVG_E_DIM;
    if (cfg > CFG_S32x64 || splits < 0) return MAVG_E_FLAG;
    return gemm_ws_floats(m, n, k, 1, cfg, splits) * 4 + 256;
}

extern "C" int32_t mavg_gemm(const float* a, int64_t lda, int32_t a_kc, const float* b, int64_t ldb, int32_t b_kc,
                             float* c, int64_t ldc, int32_t m, int32_t n, int32_t k, int32_t epi, const float* bias,
                             const float* aux, int64_t ldaux, float alpha, float beta, int32_t cfg, int32_t splits,
                             void* workspace, int64_t workspace_bytes, void* stream) {
    return mavg_gemm_parts(a, lda, a_kc, b, ldb, b_kc, c, ldc, m, n, k, epi, bias, aux, ldaux, alpha, beta, cfg, splits, MAVG_PARTS_THREE, 0, 0,
                           workspace, workspace_bytes, stream);
}

extern "C" int32_t mavg_gemm_parts(const float* a, int64_t lda, int32_t a_kc, const float* b, int64_t ldb, int32_t b_kc,
                                   float* c, int64_t ldc, int32_t m, int32_t n, int32_t k, int32_t epi, const float* bias,
                                   const float* aux, int64_t ldaux, float alpha, float beta, int32_t cfg, int32_t splits,
                                   int32_t parts, int32_t a_exp, int32_t b_exp, void* workspace, int64_t workspace_bytes, void* stream) {
    if (parts < MAVG_PARTS_THREE || parts > MAVG_PARTS_BY_DATA || a_exp < -60 || a_exp > 60 || b_exp < -60 || b_exp > 60) return MAVG_E_FLAG;
    if (!a || !b || !c) return MAVG_E_NULL;
    if (m < 1 || n < 1 || k < 0) return MAVG_E_DIM;
    if (cfg > CFG_S32x64 || splits < 0 || epi < EPI_STORE || epi > EPI_AXPBY) return MAVG_E_FLAG;
    if ((epi == EPI_BIAS || epi == EPI_BIAS_SIGMOID) && !bias) return MAVG_E_NULL;
    if (epi == EPI_MUL_DSIGMOID && !aux) return MAVG_E_NULL;
    if (lda < (a_kc ? k : m) || ldb < (b_kc ? k : n) || ldc < n || (epi == EPI_MUL_DSIGMOID && ldaux < n)) return MAVG_E_ALIGN;
    const int64_t need = gemm_ws_floats(m, n, k, 1, cfg, splits);
    if (need > 0 && (!workspace || workspace_bytes < need * 4 + 256)) return MAVG_E_WORKSPACE;
    GemmDesc g;
    g.A = a; g.lda = lda; g.a_kc = a_kc != 0;
    g.B = b; g.ldb = ldb; g.b_kc = b_kc != 0;
    g.C = c; g.ldc = ldc;
    g.M = m; g.N = n; g.K = k;
    g.epi.kind = epi; g.epi.bias = bias; g.epi.aux = aux; g.epi.ldaux = ldaux; g.epi.alpha = alpha; g.epi.beta = beta;
    g.force_cfg = cfg; g.force_splits = splits;
    g.parts = (SplitParts)parts; g.a_exp = a_exp; g.b_exp = b_exp;
    float* ws = workspace ? reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(workspace) + 255u) & ~uintptr_t(255)) : nullptr;
    return gemm_launch(g, ws, need, static_cast<hipStream_t>(stream)) == 0 ? MAVG_OK : MAVG_E_LAUNCH;
}

// Checks the problems of mavg_gemm_grouped and writes their descriptions (as many as kMaxGroups).
static int32_t grouped_descs(const mavg_gemm_problem* pr, int32_t count, int32_t a_kc, int32_t b_kc, GemmDesc* g) {
    if (!pr) return MAVG_E_NULL;
    if (count < 1 || count > kMaxGroups) return MAVG_E_DIM;
    for (int i = 0; i < count; ++i) {
        const mavg_gemm_problem& q = pr[i];
        if (!q.a || !q.b || !q.c) return MAVG_E_NULL;
        if (q.m < 1 || q.n < 1 || q.k < 0) return MAVG_E_DIM;
        if (q.epi < EPI_STORE || q.epi > EPI_AXPBY) return MAVG_E_FLAG;
        if ((q.epi == EPI_BIAS || q.epi == EPI_BIAS_SIGMOID) && !q.bias) return MAVG_E_NULL;
        if (q.epi == EPI_MUL_DSIGMOID && !q.aux) return MAVG_E_NULL;
        if (q.rowsum_dst && a_kc) return MAVG_E_FLAG;
        if (q.lda < (a_kc ? q.k : q.m) || q.ldb < (b_kc ? q.k : q.n) || q.ldc < q.n || (q.epi == EPI_MUL_DSIGMOID && q.ldaux < q.n))
            return MAVG_E_ALIGN;
        GemmDesc& d = g[i];
        d.A = q.a; d.lda = q.lda; d.a_kc = a_kc != 0;
        d.B = q.b; d.ldb = q.ldb; d.b_kc = b_kc != 0;
        d.C = q.c; d.ldc = q.ldc;
        d.M = q.m; d.N = q.n; d.K = q.k;
        d.a_pad4 = q.a_pad4 != 0; d.b_pad4 = q.b_pad4 != 0;
        d.epi.kind = q.epi; d.epi.bias = q.bias; d.epi.aux = q.aux; d.epi.ldaux = q.ldaux; d.epi.alpha = q.alpha; d.epi.beta = q.beta;
        d.epi.rowsum_dst = q.rowsum_dst; d.epi.rowsum_alpha = q.rowsum_alpha; d.epi.rowsum_beta = q.rowsum_beta;
    }
    return MAVG_OK;
}

extern "C" int32_t mavg_gemm_grouped(const mavg_gemm_problem* pr, int32_t count, int32_t a_kc, int32_t b_kc, void* stream) {
    return mavg_gemm_grouped_parts(pr, count, a_kc, b_kc, MAVG_PARTS_THREE, 0, 0, stream);
}

extern "C" int32_t mavg_gemm_grouped_parts(const mavg_gemm_problem* pr, int32_t count, int32_t a_kc, int32_t b_kc, int32_t parts, int32_t a_exp,
                                           int32_t b_exp, void* stream) {
    GemmDesc g[kMaxGroups];
    const int32_t rc = grouped_descs(pr, count, a_kc, b_kc, g);
    if (rc) return rc;
    if (parts < MAVG_PARTS_THREE || parts > MAVG_PARTS_BY_DATA || a_exp < -60 || a_exp > 60 || b_exp < -60 || b_exp > 60) return MAVG_E_FLAG;
    for (int i = 0; i < count; ++i) { g[i].parts = (SplitParts)parts; g[i].a_exp = a_exp; g[i].b_exp = b_exp; }
    return gemm_launch_grouped(g, count, static_cast<hipStream_t>(stream)) == 0 ? MAVG_OK : MAVG_E_LAUNCH;
}

extern "C" int64_t mavg_gemm_grouped_packed_bytes(const mavg_gemm_problem* pr, int32_t count) {
    GemmDesc g[kMaxGroups];
    const int32_t rc = grouped_descs(pr, count, 0, 0, g);
    if (rc) return rc;
    int64_t f = 0;
    for (int i = 0; i < count; ++i) f += gemm_packed_floats(g[i].M, g[i].N, g[i].K, 1);
    return f * 4 + 256;
}

extern "C" int32_t mavg_gemm_grouped_packed(const mavg_gemm_problem* pr, int32_t count, int32_t tiles, void* workspace, int64_t workspace_bytes, void* stream) {
    GemmDesc g[kMaxGroups];
    const int32_t rc = grouped_descs(pr, count, 0, 0, g);
    if (rc) return rc;
    if (tiles < -1 || tiles >= kPackedShapes) return MAVG_E_FLAG;
    for (int i = 0; i < count; ++i)
        if (g[i].K < 1 || g[i].epi.kind != EPI_AXPBY) return MAVG_E_FLAG;
    const int64_t need = mavg_gemm_grouped_packed_bytes(pr, count);
    if (!workspace || workspace_bytes < need) return MAVG_E_WORKSPACE;
    float* ws = reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(workspace) + 255u) & ~uintptr_t(255));
    return gemm_launch_packed(g, count, ws, need / 4 - 64, static_cast<hipStream_t>(stream), tiles) == 0 ? MAVG_OK : MAVG_E_LAUNCH;
}

extern "C" int32_t mavg_gemm_grouped_kernel(const mavg_gemm_problem* pr, int32_t count, int32_t a_kc, int32_t b_kc, int32_t which) {
    GemmDesc g[kMaxGroups];
    const int32_t rc = grouped_descs(pr, count, a_kc, b_kc, g);
    if (rc) return rc;
    if (which < 0 || which >= count) return MAVG_E_DIM;
    return gemm_grouped_kernel(g, count, which);
}
