"""The split-operand and in-workgroup-split GEMM kernels with two fp16 parts per element, as the training calls use them
(mavg_gemm_parts): what two parts hold and what they lose, values that do not survive them, and the choice between two and three parts
by the operands themselves."""
import numpy as np
import pytest

from tests.test_gpu_gemm_split_range import EXPONENTS, LAYOUTS, _check, _pick, _rows, _wide
from tests.util import dev, host, rel_err, workspace

pytestmark = pytest.mark.gpu

TWO, BY_DATA = 1, 2
CFGS = [2, 3, 4, 5, 7, 8, 9]      # split-operand tiles 256x128, 64x64, 64x128, 128x128, 32x64; in-workgroup split 32x64, 32x32


def _product(A, Bt, a_kc, b_kc, cfg, parts, splits=1, a_exp=0, b_exp=0, pad=0):
    import torch
    from paper_1507_01239_amd import binding as B
    (m, k), n = A.shape, Bt.shape[0]
    a_st, b_st = (A if a_kc else A.T), (Bt if b_kc else Bt.T)
    a_st, b_st = (np.concatenate([x, np.full((len(x), pad), np.nan, np.float32)], 1) for x in (a_st, b_st))
    c = torch.zeros(m, n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, cfg, splits))
    B.mavg_gemm_parts(dev(a_st), a_st.shape[1], a_kc, dev(b_st), b_st.shape[1], b_kc, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, cfg, splits,
                      parts, a_exp, b_exp, ws)
    torch.cuda.synchronize()
    return host(c).astype(np.float64)


def _ref(A, Bt):
    return A.astype(np.float64) @ Bt.astype(np.float64).T


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("parts", [TWO, BY_DATA])
def test_tile_edges_and_contraction_remainders(parts, cfg, a_kc, b_kc):
    # m, n at tile edges; one k-tile to many, with and without a partial one, fewer tiles than k-groups; rows aligned to 4 bytes only
    # (the in-workgroup-split kernels: 16, or another kernel runs).  Tolerance: every addition of 1040 rounding by 2^-24 gives 1.4e-6.
    rng = np.random.default_rng(300 + cfg)
    for m, n, k, pad in [(1, 1, 16, 0), (255, 129, 17, 0), (128, 128, 31, 1), (257, 127, 32, 3), (33, 65, 47, 0), (300, 200, 63, 2), (64, 64, 64, 0),
                         (200, 132, 128, 0), (65, 200, 96, 0), (260, 140, 140, 0), (256, 256, 143, 1), (132, 72, 1040, 0)]:
        A, Bt = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((n, k)).astype(np.float32)
        assert rel_err(_product(A, Bt, a_kc, b_kc, cfg, parts, pad=pad), _ref(A, Bt)) < 2e-6, (m, n, k, pad)
    A, Bt = rng.standard_normal((270, 700)).astype(np.float32), rng.standard_normal((133, 700)).astype(np.float32)
    assert rel_err(_product(A, Bt, a_kc, b_kc, cfg, parts, splits=3), _ref(A, Bt)) < 2e-6


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("parts", [TWO, BY_DATA])
@pytest.mark.parametrize("k", [76, 268])
def test_rows_of_any_magnitude(parts, cfg, a_kc, b_kc, k):
    # every row within 2^8 of its largest element: as close as float32 products, whatever that element is (and two groups of ordinary rows)
    rng = np.random.default_rng(310 + cfg)
    m, n = 152, 140
    A, Bt = _rows(rng, m, k, EXPONENTS), _rows(rng, n, k, [e for e in EXPONENTS if e is None or e < 80])
    A[64:128], Bt[32:64] = _rows(rng, 64, k, [-14, 0, 15]), _rows(rng, 32, k, [-14, 0, 15])
    _check(_product(A, Bt, a_kc, b_kc, cfg, parts), A, Bt)


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", CFGS)
def test_what_two_parts_lose(cfg, a_kc, b_kc):
    # Elements over 60 powers of two, rows whose largest is about 1: 2^-36 of an element may be lost, times the other factors, beside
    # the 2^-21 of each product (and the additions').  Scaled by 2^10, 2^-46.
    rng = np.random.default_rng(320 + cfg)
    m, n, k = 152, 140, 268
    A, Bt = _wide(rng, m, k, -60, 0), _wide(rng, n, k, -60, 0)
    A[:, ::16] = rng.uniform(0.5, 1, (m, len(range(0, k, 16))))
    Bt[:, 5::16] = rng.uniform(0.5, 1, (n, len(range(5, k, 16))))
    A64, B64 = np.abs(A.astype(np.float64)), np.abs(Bt.astype(np.float64))
    for e in (0, 10):
        got = _product(A, Bt, a_kc, b_kc, cfg, TWO, a_exp=e, b_exp=e)
        fa, fb = (0 if a_kc and b_kc else e), (e if not a_kc and not b_kc else 0)      # (what is scaled)
        bound = 1.5e-6 * (A64 @ B64.T) + 2.0 ** (-36 - fa) * B64.sum(1)[None] + 2.0 ** (-36 - fb) * A64.sum(1)[:, None]
        assert (np.abs(got - _ref(A, Bt)) <= bound).all()


@pytest.mark.parametrize("cfg", CFGS)
def test_single_products(cfg):
    # One term per sum, the others zero (with ordinary values in either operand, or the kernels would not take two parts).  Of 1 + 2^-11 +
    # 2^-23 the high part rounds up to 1 + 2^-10, the low one (4095 units) to 4096, and the product of two low parts, 2^-22, is left
    # out: three errors of one sign, 2^-21 in all, the most there is, and two additions.  That two parts did it shows in the error; with
    # three parts (or float32 products) there are 2^-24 left out at most and five additions.
    rng = np.random.default_rng(330)
    m = n = 64
    k = 128
    x = (1 + rng.integers(0, 2 ** 23, m) * 2.0 ** -23).astype(np.float32)
    x[:32] = 1 + 2.0 ** -11 + 2.0 ** -23
    A, Bt = np.zeros((m, k), np.float32), np.zeros((n, k), np.float32)
    A[:, 0] = Bt[:, 0] = x
    A[:, 2::16] = A[:, 5::16] = Bt[:, 3::16] = Bt[:, 6::16] = 1
    ref = x[:, None].astype(np.float64) * x[None]
    err = np.abs(_product(A, Bt, 1, 1, cfg, TWO) - ref) / ref
    assert err.max() <= 2.0 ** -21 + 2.0 ** -23 and err[:32, :32].max() > 2.0 ** -22
    assert (np.abs(_product(A, Bt, 1, 1, cfg, 0) - ref) <= 6 * 2.0 ** -24 * ref).all()


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("parts", [0, TWO, BY_DATA])
def test_values_that_do_not_survive_the_parts(parts, cfg, a_kc, b_kc):
    # infinities, NaNs and floats too large for either, in the first k-group's share, in others', and in the rest of the contraction
    rng = np.random.default_rng(340)
    m, n, k = 100, 140, 268
    A, Bt = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((n, k)).astype(np.float32)
    A[3, 5], A[40, 267], A[41, 77], A[70, 0], A[71, 130], A[97, 200] = np.inf, np.nan, np.nan, 3.4e38, -np.inf, 1e6
    Bt[:, 0] = 1e-3 * np.abs(Bt[:, 0])       # 3.4e38 * 1e-3 stays finite
    Bt[9, 5] = 0.0                           # inf * 0
    Bt[77, 5], Bt[130, 265] = -np.inf, np.inf
    got = _product(A, Bt, a_kc, b_kc, cfg, parts)
    with np.errstate(all="ignore"):
        ref = (A.astype(np.float64)[:, None, :] * Bt.astype(np.float64)[None]).sum(axis=2)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf])
    fine = np.isfinite(ref)
    assert np.isfinite(got[fine]).all()
    rows = np.repeat(np.arange(m)[:, None], n, 1)
    for r in (70, 97):
        assert rel_err(got[fine & (rows == r)], ref[fine & (rows == r)]) < 2e-6
    rest = fine & (rows != 70) & (rows != 97)
    assert rel_err(got[rest], ref[rest]) < 2e-6


@pytest.mark.parametrize("m,n,k", [(1024, 2048, 2048), (256, 2048, 2048)])
def test_long_sums_of_ordinary_terms_are_closer_than_float32_products(m, n, k):
    rng = np.random.default_rng(350)
    A, Bt = rng.random((m, k), dtype=np.float32), rng.standard_normal((n, k), dtype=np.float32)
    import torch
    ref = (dev(A).double() @ dev(Bt).double().T).cpu().numpy()
    assert rel_err(_product(A, Bt, 1, 1, -1, TWO, splits=0), ref) < 0.5 * rel_err(_product(A, Bt, 1, 1, 0, TWO), ref)


@pytest.mark.parametrize("parts", [TWO, BY_DATA])
@pytest.mark.parametrize("n,shapes,kernel", [(101, [(1155, 1537), (130, 65)], 0), (263, [(4100, 4100), (130, 68)], 0)])
def test_grouped_updates(parts, n, shapes, kernel):
    # ordinary values and rows of any magnitude, in one launch with a small problem beside the large one; row sums
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(360)
    for exps in (None, EXPONENTS):
        probs, keep = [], []
        for (m, nc) in shapes:
            ldd = (m + 3) // 4 * 4 if n > 200 else m
            D = np.zeros((n, ldd), np.float32)
            D[:, :m] = rng.standard_normal((n, m)) if exps is None else _rows(rng, m, n, exps).T
            X = (rng.standard_normal((n, nc)) if exps is None else _rows(rng, nc, n, [e for e in exps if e is None or e < 80]).T).astype(np.float32)
            W, bv = np.zeros((m, nc), np.float32), np.zeros(m, np.float32)
            if exps is None: W, bv = rng.standard_normal((m, nc)).astype(np.float32), rng.standard_normal(m).astype(np.float32)
            t = [dev(v) for v in (D, X, W, bv)]
            probs.append(B.gemm_problem(t[0], ldd, t[1], nc, t[2], nc, m, nc, n, epi=4, alpha=-0.25, beta=1.0, rowsum_dst=t[3], rowsum_alpha=-0.25,
                                        rowsum_beta=1.0, a_pad4=ldd != m))
            keep.append((t, D[:, :m], X, W, bv))
        assert B.mavg_gemm_grouped_kernel(probs, 0, 0, 0) == kernel
        B.mavg_gemm_grouped_parts(probs, 0, 0, parts, 0, 0)
        torch.cuda.synchronize()
        for t, D, X, W, bv in keep:
            if exps is None:
                assert rel_err(host(t[2]), W - 0.25 * _ref(D.T, X.T)) < 2e-6
                assert rel_err(host(t[3]), bv - 0.25 * D.astype(np.float64).sum(axis=0)) < 2e-6
            else:
                _check(-4.0 * host(t[2]).astype(np.float64), D.T, X.T)


@pytest.mark.parametrize("parts", [TWO, BY_DATA])
def test_grouped_updates_in_256x128_tiles(parts):
    # from 1024 rows and 32 tiles of 128x128 per compute unit on; ragged tile edges, a partial k-tile, row sums, a small problem beside.
    # Tolerance: every addition of 1027 rounding by 2^-24 gives 1.4e-6.
    import torch
    from paper_1507_01239_amd import binding as B
    n, probs, keep = 1027, [], []
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    for (m, nc) in [(8196, 16300), (130, 68), (513, 259)]:
        ldd = (m + 3) // 4 * 4
        t = [torch.randn(s, generator=g, device="cuda") for s in ((n, ldd), (n, nc), (m, nc), (m,))]
        ref = (t[2].double() - 0.25 * (t[0][:, :m].double().T.contiguous() @ t[1].double()), t[3].double() - 0.25 * t[0][:, :m].double().sum(0))
        probs.append(B.gemm_problem(t[0], ldd, t[1], nc, t[2], nc, m, nc, n, epi=4, alpha=-0.25, beta=1.0, rowsum_dst=t[3], rowsum_alpha=-0.25,
                                    rowsum_beta=1.0, a_pad4=True))
        keep.append((t, ref))
    assert [B.mavg_gemm_grouped_kernel(probs, 0, 0, i) for i in range(3)] == [0, 0, 0]
    B.mavg_gemm_grouped_parts(probs, 0, 0, parts, 5, 5)
    torch.cuda.synchronize()
    for t, (Wr, br) in keep:
        for got, ref in ((t[2], Wr), (t[3], br)):
            assert ((got.double() - ref).norm() / ref.norm()).item() < 2e-6


def test_arguments():
    import torch
    from paper_1507_01239_amd import binding as B
    x = torch.zeros(64, 64, device="cuda")
    for parts, ea, eb in [(-1, 0, 0), (3, 0, 0), (1, 61, 0), (1, 0, -61)]:
        with pytest.raises(B.MavgError) as e:
            B.mavg_gemm_parts(x, 64, 1, x, 64, 1, torch.zeros_like(x), 64, 64, 64, 64, 0, None, None, 0, 1.0, 0.0, -1, 1, parts, ea, eb, None)
        assert e.value.code == B.E_FLAG
        with pytest.raises(B.MavgError) as e:
            B.mavg_gemm_grouped_parts([B.gemm_problem(x, 64, x, 64, torch.zeros_like(x), 64, 64, 64, 64)], 0, 0, parts, ea, eb)
        assert e.value.code == B.E_FLAG


# ---- two parts or three, as the operands ask for ----------------------------------------------------------------------------------------


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("cfg", CFGS)
def test_rows_that_begin_small_lose_nothing(cfg, a_kc, b_kc):
    # nothing but small elements to begin with and large ones later, facing zeros: three parts (in the in-workgroup-split kernels,
    # float32 products), exact as mavg_gemm is
    rng = np.random.default_rng(370 + cfg)
    m, n, k = 300, 152, 268
    A = _wide(rng, m, k, -80, -40)
    late = rng.integers(130, k, m)
    A[np.arange(m), late] = rng.uniform(0.5, 1, m)
    Bt = np.maximum(_pick(rng, n, k, rng.integers(0, 120, n)), 2.0 ** -12 * (np.arange(k) < 130)).astype(np.float32)
    _check(_product(A, Bt, a_kc, b_kc, cfg, BY_DATA), A, Bt)


@pytest.mark.parametrize("cfg", [2, 3, 4, 5, 9])
@pytest.mark.parametrize("m,n,k,splits", [(1, 1, 17, 1), (257, 129, 40, 1), (300, 140, 700, 3), (33, 65, 1201, 1)])
def test_one_small_row_among_many(cfg, m, n, k, splits):
    # one row far below the others, in the last tile; a contraction of a partial k-tile and one whole one, and in splits
    rng = np.random.default_rng(380)
    A, Bt = rng.uniform(0.5, 2, (m, k)).astype(np.float32), rng.uniform(0.5, 2, (n, k)).astype(np.float32)
    A[m - 1] *= np.float32(2.0 ** -50)
    for a_kc, b_kc in ((1, 0), (0, 0)):
        _check(_product(A, Bt, a_kc, b_kc, cfg, BY_DATA, splits), A, Bt)
        _check(_product(Bt, A, a_kc, b_kc, cfg, BY_DATA, splits), Bt, A)


def _graph_us(calls):
    """Microseconds a call of each of `calls`, captured twenty times over in a graph each and replayed in turn."""
    import torch
    graphs = []
    for f in calls:
        f()
        torch.cuda.synchronize()
        g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(g, stream=s):
            for _ in range(20):
                f()
        graphs.append(g)
    best = [1e9] * len(calls)
    for _ in range(12):
        for i, g in enumerate(graphs):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            g.replay()
            e1.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], e0.elapsed_time(e1) * 50)
    return best


def test_small_rows_take_no_multiple_of_the_time():
    # one class in 32 whose errors are all far below the others', as with a trained network and thousands of classes: measured 1.3 times
    # the time of ordinary errors (4.1 times when their blocks go to the fp32 matrix cores, as with MAVG_PARTS_TWO)
    import torch
    from paper_1507_01239_amd import binding as B
    n, m, nc = 512, 8000, 2048
    d, x, w = torch.randn(n, m, device="cuda"), torch.rand(n, nc, device="cuda"), torch.zeros(m, nc, device="cuda")
    small = d.clone()
    small[:, ::32] *= 2.0 ** -50
    call = lambda t, parts=BY_DATA: lambda: B.mavg_gemm_grouped_parts([B.gemm_problem(t, m, x, nc, w, nc, m, nc, n, epi=4, alpha=1e-6, beta=1.0)], 0, 0, parts, 0, 0)
    assert B.mavg_gemm_grouped_kernel([B.gemm_problem(d, m, x, nc, w, nc, m, nc, n, epi=4, alpha=1e-6, beta=1.0)], 0, 0, 0) == 0
    ordinary, with_small, recomputed = _graph_us([call(d), call(small), call(small, TWO)])
    assert with_small < 1.5 * ordinary, (ordinary, with_small, recomputed)


@pytest.mark.parametrize("m,n,k", [(145, 145, 129), (77, 501, 129), (200, 1021, 150)])
def test_short_ragged_products_take_no_longer_with_two_parts(m, n, k):
    # 8.4 against 7.9 us when they went to the kernels with two parts
    import torch
    from paper_1507_01239_amd import binding as B
    a, b, c = torch.rand(m * k, device="cuda"), torch.randn(n * k, device="cuda"), torch.empty(m * n, device="cuda")
    ws = workspace(B.mavg_gemm_workspace_bytes(m, n, k, -1, 0))
    call = lambda parts: lambda: B.mavg_gemm_parts(a, k, 1, b, n, 0, c, n, m, n, k, 0, None, None, 0, 1.0, 0.0, -1, 0, parts, 5, 5, ws)
    three, two, by_data = _graph_us([call(0), call(TWO), call(BY_DATA)])
    assert two < 1.04 * three and by_data < 1.04 * three, (three, two, by_data)


@pytest.mark.parametrize("a_kc,b_kc", LAYOUTS)
@pytest.mark.parametrize("m,n,k", [(513, 1020, 512), (65, 8132, 516), (1024, 1024, 2304), (100, 5188, 1000), (2052, 196, 1337), (832, 640, 576), (576, 1000, 2060),
                                   (1024, 2048, 512), (4161, 260, 533), (769, 1928, 1100), (130, 8196, 1020), (33, 24576, 517), (770, 2048, 2304),
                                   (594, 2768, 2389), (190, 4480, 2485), (130, 2512, 4816), (1, 6160, 4805)])
def test_64x64_and_64x128_tiles_split_inside_the_workgroup(m, n, k, a_kc, b_kc):
    # 129 to 256 tiles of 64x64, and 192 to 256 of 64x128, the shortest and longest contractions that go there, remainders of k-tiles (4, 5, 8, 9, 12
    # steps), numbers of k-tiles that four wavefronts share unevenly, and partial tiles; an odd k by row strides.  Tolerance: 2304 additions
    # rounding by 2^-24 each give 3e-6 if all round alike, 2e-7 if they round at random.  The last four, with n-contiguous B: longer ones, unsplit and split
    # across workgroups in two and four.
    import torch
    from paper_1507_01239_amd import binding as B
    rng = np.random.default_rng(m + k)
    whole = 4 if -(-m // 64) * -(-n // 64) <= 256 else 16      # (rows that do not begin at 16, or 64, bytes go elsewhere)
    m, n = m if a_kc else -(-m // whole) * whole, n if b_kc else -(-n // whole) * whole
    A, Bt = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((n, k)).astype(np.float32)
    pad = -k % whole
    stored = [np.pad(x, ((0, 0), (0, pad)), constant_values=np.nan) if kc else x.T for x, kc in ((A, a_kc), (Bt, b_kc))]
    a, b = dev(np.ascontiguousarray(stored[0])), dev(np.ascontiguousarray(stored[1]))
    bias = rng.standard_normal(n).astype(np.float32)

    def run(epi, a=a, b=b):
        c = torch.full((m, n + 4), 7.0, device="cuda")
        B.mavg_gemm_parts(a, a.shape[1], a_kc, b, b.shape[1], b_kc, c, n + 4, m, n, k, epi, dev(bias), None, 0, 1.0, 0.0, -1, 0, TWO, 0, 0,
                          workspace(B.mavg_gemm_workspace_bytes(m, n, k)))
        assert (c[:, n:] == 7.0).all()
        return host(c)[:, :n].astype(np.float64)
    want = _ref(A, Bt)
    first = run(0)
    assert rel_err(first, want) < 4e-7
    assert rel_err(run(2), 1 / (1 + np.exp(-want - bias))) < 2e-6      # (sigmoid: sums of magnitude 40 off by 2e-7 of that)
    assert np.array_equal(first, run(0))
    # one block of rows with an infinity, one with a NaN, one of nothing but small elements, and the others as before
    hurt = a.clone()
    rows = (lambda i: hurt[i]) if a_kc else (lambda i: hurt[:, i])
    rows(0)[k - 1], rows(m // 2)[1] = float("inf"), float("nan")
    if m > 200:
        rows(m - 1)[:k] *= 2.0**-60
    got, ref = run(0, a=hurt), (hurt[:, :k] if a_kc else hurt.T).double().cpu().numpy() @ Bt.astype(np.float64).T
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    fine = np.isfinite(ref).all(1)
    assert (np.linalg.norm(got[fine] - ref[fine], axis=1) <= 2e-6 * np.linalg.norm(ref[fine], axis=1)).all()
