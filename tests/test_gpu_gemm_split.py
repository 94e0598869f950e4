"""The split-operand GEMM kernels (three bf16 parts per float32 element) against float64 products of the same float32
inputs, at the sizes where they can go wrong, and with values that do not survive the split."""
import numpy as np
import pytest

from tests.test_gpu_gemm import _run
from tests.util import dev, host, rel_err, workspace

pytestmark = pytest.mark.gpu

LAYOUTS = [(1, 1), (1, 0), (0, 0), (0, 1)]
SPLIT_CFGS = [3, 4, 5, 9]      # 64x64, 64x128, 128x128, 32x64 tiles


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", SPLIT_CFGS)
def test_tile_edges_and_contraction_remainders(a_kc, b_kc, cfg):
    # m and n one below, at and above the tiles' edges; contractions of one to many 16-step tiles, with and without a
    # partial one, fewer tiles than k-groups, shares that end in a partial tile; rows aligned to 4 bytes only.
    # Tolerance: a product of k terms of random sign is off by about 2^-24 sqrt(k / 2) where every addition rounds;
    # k = 1040 gives 1.4e-6, and the k-groups add in parts.
    for i, (m, n, k, pad) in enumerate([(1, 1, 16, 0), (127, 129, 17, 0), (128, 128, 31, 1), (129, 127, 32, 3), (33, 65, 33, 0),
                                        (31, 63, 48, 2), (64, 64, 63, 0), (200, 130, 79, 1), (65, 200, 128, 0), (130, 70, 1040, 1)]):
        assert _run(m, n, k, a_kc, b_kc, cfg=cfg, seed=100 + i, pad=pad) < 2e-6, (m, n, k, pad)
    assert _run(70, 133, 700, a_kc, b_kc, cfg=cfg, splits=3, seed=120, epi=2, alpha=-0.5) < 2e-6
    assert _run(70, 133, 15, a_kc, b_kc, cfg=cfg, seed=121) < 2e-6      # below one k-tile: another kernel runs


@pytest.mark.parametrize("epi", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("cfg", SPLIT_CFGS)
def test_epilogues(epi, cfg):
    assert _run(150, 200, 90, 1, 1, epi=epi, cfg=cfg, seed=130, alpha=-0.5, beta=1.0) < 2e-6
    assert _run(150, 201, 90, 0, 0, epi=epi, cfg=cfg, seed=131, alpha=0.25, beta=0.5, pad=1) < 2e-6


@pytest.mark.parametrize("cfg", SPLIT_CFGS)
def test_single_products_where_the_second_part_rounds_up(cfg):
    # One term per sum, of factors 1 + 2^-8 - j 2^-23: h = 1, m = 2^-8, l = -j 2^-23, and the six products that are kept add
    # up without rounding.  What is left out is (i + j) 2^-31 + i j 2^-46, below 2^-24 for i, j <= 60; with a second part cut
    # off instead of rounded it would be 2^-23.
    import torch
    from paper_1507_01239_amd import binding as B
    m, n, k = 60, 60, 16
    x = (1 + 2.0 ** -8 - np.arange(1, 61) * 2.0 ** -23).astype(np.float32)
    A = np.zeros((m, k), np.float32)
    A[np.arange(m), np.arange(m) % k] = x
    c = torch.zeros(m, n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, cfg, 1))
    B.mavg_gemm(dev(A), k, 1, dev(np.repeat(x[:, None], k, 1)), k, 1, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, 1, ws)
    torch.cuda.synchronize()
    ref = x[:, None].astype(np.float64) * x[None]
    assert (np.abs(host(c) - ref) <= 2.0 ** -24 * ref).all()


@pytest.mark.parametrize("cfg", SPLIT_CFGS)
def test_values_that_do_not_survive_the_split(cfg):
    # infinities, NaNs and floats that round to infinity in bf16 give what float32 arithmetic gives; rows and columns
    # without them are untouched
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(7)
    m, n, k = 100, 140, 120
    A, Bt = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((n, k)).astype(np.float32)
    A[3, 5], A[40, 119], A[70, 0], A[71, 1] = np.inf, np.nan, 3.4e38, -np.inf
    Bt[:, 0] = 1e-3 * np.abs(Bt[:, 0])       # 3.4e38 * 1e-3 stays finite
    Bt[9, 5] = 0.0                           # inf * 0
    Bt[77, 5] = -np.inf
    c = torch.zeros(m, n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, cfg, 1))
    B.mavg_gemm(dev(A), k, 1, dev(Bt), k, 1, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, 1, ws)
    torch.cuda.synchronize()
    got = host(c).astype(np.float64)
    with np.errstate(all="ignore"):
        ref = (A.astype(np.float64)[:, None, :] * Bt.astype(np.float64)[None]).sum(axis=2)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf])
    fine = np.isfinite(ref)
    assert np.isfinite(got[fine]).all()
    big = fine & (np.arange(m)[:, None] == 70)
    assert rel_err(got[big], ref[big]) < 2e-6
    assert rel_err(got[fine & ~big], ref[fine & ~big]) < 2e-6


@pytest.mark.parametrize("k,pad", [(16, 0), (72, 1), (264, 3), (640, 0)])
@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", SPLIT_CFGS)
def test_blocks_with_a_non_finite_value_are_recomputed(cfg, a_kc, b_kc, k, pad):
    # one infinity in the first operand: its row is infinite or NaN, and the rows that are recomputed beside it are float32
    # products as before; every layout, contractions with and without a partial k-tile, fewer k-tiles than k-groups and more
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(70 + k)
    m, n, lda, ldb = 70, 150, (k if a_kc else 70) + pad, (k if b_kc else 150) + pad
    A, Bm = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((k, n)).astype(np.float32)
    A[37, k - 1] = np.inf
    a_st, b_st = np.zeros((m if a_kc else k, lda), np.float32), np.zeros((n if b_kc else k, ldb), np.float32)
    a_st[:, :k if a_kc else m] = A if a_kc else A.T
    b_st[:, :k if b_kc else n] = Bm.T if b_kc else Bm
    c = torch.zeros(m, n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, cfg, 1))
    B.mavg_gemm(dev(a_st), lda, a_kc, dev(b_st), ldb, b_kc, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, 1, ws)
    torch.cuda.synchronize()
    got = host(c)
    assert np.array_equal(got[37], np.where(Bm[k - 1] > 0, np.inf, -np.inf).astype(np.float32))
    rows = np.arange(m) != 37
    assert rel_err(got[rows], (A[rows].astype(np.float64) @ Bm.astype(np.float64))) < 2e-6


def test_a_product_of_nothing_but_nans_takes_no_multiple_of_its_time():
    # every block recomputed: measured 2.9 times the time of ordinary values (8 times with dependent single loads)
    import torch
    from paper_1507_01239_amd import binding as B
    m, n, k = 1024, 2048, 2048
    b, c = torch.randn(n, k, device="cuda"), torch.empty(m, n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, 4, 1))

    def best_ms(a):
        t = []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                B.mavg_gemm(a, k, 1, b, k, 1, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, 4, 1, ws)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
        return min(t)
    ordinary = best_ms(torch.rand(m, k, device="cuda"))
    assert best_ms(torch.full((m, k), float("nan"), device="cuda")) < 5 * ordinary


# Elements whose parts bf16 cannot hold (below 2^-110 the third one, at 2^-132 all but one bit): float32 products all the same.
# The second scale keeps the results above the float32 denormals, whose rounding the tolerance does not cover.
@pytest.mark.parametrize("scale,other", [(1e-30, 1.0), (1e-34, 1.0), (1e-36, 1.0), (1e-38, 1e6), (1e-40, 1e10)])
@pytest.mark.parametrize("cfg", SPLIT_CFGS)
def test_small_magnitudes(cfg, scale, other):
    rng = np.random.default_rng(8)
    m, n, k = 70, 90, 64
    A = (rng.uniform(1, 2, (m, k)) * scale).astype(np.float32)
    Bt = (rng.standard_normal((n, k)) * other).astype(np.float32)
    import torch
    from paper_1507_01239_amd import binding as B
    c = torch.zeros(m, n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, cfg, 1))
    B.mavg_gemm(dev(A), k, 1, dev(Bt), k, 1, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, 1, ws)
    torch.cuda.synchronize()
    assert rel_err(host(c), A.astype(np.float64) @ Bt.astype(np.float64).T) < 2e-6


# Few rows over a long contraction, few columns, about one tile per compute unit: where the split-operand kernels lose.
@pytest.mark.parametrize("m,n,k,a_kc,b_kc", [(64, 2048, 8000, 1, 0), (96, 624, 6064, 0, 0), (3329, 175, 1036, 1, 1), (32, 3200, 1728, 1, 0)])
def test_automatic_plans_are_not_slower_than_the_fp32_kernels(m, n, k, a_kc, b_kc):
    # up to 1.3 times the time of cfg 0 when they went to a split-operand kernel; 1.1 leaves room for the clock
    import torch
    from paper_1507_01239_amd import binding as B
    a, b, c = torch.rand(m * k, device="cuda"), torch.randn(n * k, device="cuda"), torch.empty(m, n, device="cuda")
    ws = workspace(max(B.mavg_gemm_workspace_bytes(m, n, k, cfg, 0) for cfg in (-1, 0)))
    best = {-1: 1e9, 0: 1e9}
    for rep in range(12):
        for cfg in best:
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                B.mavg_gemm(a, k if a_kc else m, a_kc, b, k if b_kc else n, b_kc, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, 0, ws)
            e1.record()
            torch.cuda.synchronize()
            best[cfg] = min(best[cfg], e0.elapsed_time(e1))
    assert best[-1] < 1.1 * best[0], best


@pytest.mark.parametrize("k", [16, 24, 31, 32, 48, 79, 80, 96])
def test_short_contractions_are_no_less_exact_than_with_fp32_products(k):
    # positive terms, ragged rows, a problem large enough for the split-operand kernels: their sums of one k-tile are off by up
    # to 1.4 times as much as those of the float32 kernel (cfg 1), the grouped launch's up to 1.4 times at 16 and 1.2 times at
    # 32 steps, so the float32 kernels run there (2 %: the order of their sums)
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(90 + k)
    m, n = 1003, 2001
    A, Bt = rng.random((m, k), dtype=np.float32), rng.random((n, k), dtype=np.float32)
    ref = A.astype(np.float64) @ Bt.astype(np.float64).T
    err = []
    for cfg in (-1, 1):
        c = torch.zeros(m, n, device="cuda")
        ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, cfg, 0))
        B.mavg_gemm(dev(A), k, 1, dev(Bt), k, 1, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, 0, ws)
        torch.cuda.synchronize()
        err.append(rel_err(host(c), ref))
    # the same product as a grouped update of zeros
    c = torch.zeros(m, n, device="cuda")
    B.mavg_gemm_grouped([B.gemm_problem(dev(A.T.copy()), m, dev(Bt.T.copy()), n, c, n, m, n, k, epi=4, alpha=1.0, beta=1.0)], 0, 0)
    torch.cuda.synchronize()
    err.append(rel_err(host(c), ref))
    assert err[0] <= 1.02 * err[1] and err[2] <= 1.02 * err[1], err


# Weight updates C <- C - 0.25 D^T A with row sums, several in one launch: (rows n, shapes, kernel of each problem: 0 =
# split-operand, 1 = direct-to-LDS, 2 = register-staged).  Ragged tile edges, whole and partial k-tiles, small problems
# next to a large one; aligned problems need 1024 tiles of 128x128 (512 from 520 rows on), ragged ones 128, and both enough rows.
# Tolerance: a product of n terms of random sign is off by about 2^-24 sqrt(n / 2) where every addition rounds: 1e-6 at 520.
BIG, HALF, SMALL, RAGGED = (4100, 4100), (2052, 4100), [(130, 68), (514, 260)], [(1027, 1537), (130, 65), (514, 259)]


@pytest.mark.parametrize("n,shapes,kernels", [
    (16, [(1027, 1540)] + SMALL, [1, 1, 1]), (200, [BIG] + SMALL, [0, 0, 0]), (263, [BIG] + SMALL, [0, 0, 0]),
    (263, [(1027, 1540)] + SMALL, [1, 1, 1]), (520, [HALF] + SMALL, [0, 0, 0]),
    (16, RAGGED, [2, 2, 2]), (79, RAGGED, [2, 2, 2]), (80, RAGGED, [0, 0, 0]), (200, RAGGED, [0, 0, 0]), (263, RAGGED, [0, 0, 0]),
    # aligned and ragged problems in one call: on one kernel, on two
    (263, [BIG, (514, 259), (130, 68)], [0, 0, 0]), (100, [(1027, 1540), (514, 259), (130, 68)], [1, 0, 1]),
    (30, [(514, 260), (514, 259)], [1, 2])])
def test_grouped_weight_updates(n, shapes, kernels):
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(50 + n)
    probs, refs, outs, keep = [], [], [], []
    for (m, nc) in shapes:
        ldd = (m + 3) // 4 * 4
        D = np.zeros((n, ldd), np.float32)
        D[:, :m] = rng.standard_normal((n, m))
        A, W, bv = (rng.standard_normal(s).astype(np.float32) for s in ((n, nc), (m, nc), (m,)))
        d_d, a_d, w_d, b_d = dev(D), dev(A), dev(W), dev(bv)
        probs.append(B.gemm_problem(d_d, ldd, a_d, nc, w_d, nc, m, nc, n, epi=4, alpha=-0.25, beta=1.0, rowsum_dst=b_d,
                                    rowsum_alpha=-0.25, rowsum_beta=1.0, a_pad4=True))
        refs.append((W - 0.25 * D[:, :m].astype(np.float64).T @ A.astype(np.float64), bv - 0.25 * D[:, :m].astype(np.float64).sum(axis=0)))
        outs.append((w_d, b_d))
        keep.append((d_d, a_d))
    assert [B.mavg_gemm_grouped_kernel(probs, 0, 0, i) for i in range(len(probs))] == kernels
    B.mavg_gemm_grouped(probs, 0, 0)
    torch.cuda.synchronize()
    for (w_d, b_d), (Wr, br) in zip(outs, refs):
        assert rel_err(host(w_d), Wr) < 2e-6 and rel_err(host(b_d), br) < 2e-6


@pytest.mark.parametrize("kind", ["infinity", "small"])
def test_grouped_updates_with_an_infinity_and_with_small_values(kind):
    # the grouped kernel recomputes blocks as the others do: one infinite error makes one row of the update infinite, errors
    # of 1e-36 count in full (C is zero before)
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(81)
    n, m, nc, ld = 101, 1155, 1537, 1156
    D, A = rng.standard_normal((n, ld)).astype(np.float32), (1 + rng.random((n, nc))).astype(np.float32)
    if kind == "small": D *= np.float32(1e-36)
    else: D[n - 1, 700] = np.inf
    c, b, d_d, a_d = torch.zeros(m, nc, device="cuda"), torch.zeros(m, device="cuda"), dev(D), dev(A)
    prob = [B.gemm_problem(d_d, ld, a_d, nc, c, nc, m, nc, n, epi=4, alpha=1.0, beta=1.0, rowsum_dst=b, rowsum_alpha=1.0, rowsum_beta=1.0, a_pad4=True)]
    assert B.mavg_gemm_grouped_kernel(prob, 0, 0, 0) == 0
    B.mavg_gemm_grouped(prob, 0, 0)
    torch.cuda.synchronize()
    got, sums, rows = host(c), host(b), np.arange(m)
    if kind == "infinity":
        assert np.isposinf(got[700]).all() and np.isposinf(sums[700])
        rows = np.delete(rows, 700)
    Dr = D[:, rows].astype(np.float64)
    assert rel_err(got[rows], Dr.T @ A.astype(np.float64)) < 2e-6 and rel_err(sums[rows], Dr.sum(axis=0)) < 2e-6
