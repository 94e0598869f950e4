"""Weight updates on packed operands (mavg_gemm_grouped_packed): every tile shape and form of the packing launch, at the edges of tiles,
k-tiles and column groups, against float64 products."""
import numpy as np
import pytest
import torch

from paper_1507_01239_amd import binding as B

pytestmark = pytest.mark.gpu


def _problem(rng, n, m, c, pad=0, scale_a=None):
    a = rng.standard_normal((n, m)).astype(np.float32)
    if scale_a is not None:
        a = np.ldexp(a, scale_a(m)[None, :]).astype(np.float32)
    b = rng.random((n, c)).astype(np.float32)
    return a, b


def _dev(x, ld):
    t = torch.full((x.shape[0], ld), float("nan"), device="cuda")      # (the padding is never read into a result)
    t[:, :x.shape[1]] = torch.from_numpy(x).cuda()
    return t


def _update(ops, tiles, c0=0.0, bias=True):
    """C = c0 + A^T B of every pair (A, B), and the column sums of A, on the device."""
    keep, probs, outs, sums = [], [], [], []
    for a, b in ops:
        n, m, c = a.shape[0], a.shape[1], b.shape[1]
        da, db = _dev(a, m + 3), _dev(b, c + 1)
        out = torch.full((m, c), c0, device="cuda")
        s = torch.zeros(m, device="cuda")
        keep += [da, db]
        outs.append(out)
        sums.append(s)
        probs.append(B.gemm_problem(da, m + 3, db, c + 1, out, c, m, c, n, epi=4, alpha=1.0, beta=1.0,
                                    rowsum_dst=s if bias else None, rowsum_alpha=1.0, rowsum_beta=1.0))
    ws = torch.empty(B.mavg_gemm_grouped_packed_bytes(probs), dtype=torch.uint8, device="cuda")
    B.mavg_gemm_grouped_packed(probs, tiles, ws)
    torch.cuda.synchronize()
    return [o.cpu().numpy().astype(np.float64) for o in outs], [s.cpu().numpy().astype(np.float64) for s in sums]


def _check(a, b, got, sums):
    a, b = a.astype(np.float64), b.astype(np.float64)
    ref, mags = a.T @ b, np.abs(a).T @ np.abs(b)
    # a product is off by 2^-21 at most; a sum has two roundings of the accumulators per 16 steps, and three at the end
    bound = (2.0 ** -21 + (a.shape[0] / 8 + 3) * 2.0 ** -24) * mags + 2.0 ** -149
    assert (np.abs(got - ref) <= bound).all()
    assert np.linalg.norm(got - ref) <= 3e-7 * np.linalg.norm(mags)
    s = a.sum(0)
    assert (np.abs(sums - s) <= a.shape[0] * 2.0 ** -24 * np.abs(a).sum(0) + 2.0 ** -149).all()


@pytest.mark.parametrize("tiles", [-1, 0, 1, 2])
@pytest.mark.parametrize("n", [1, 15, 17, 64, 80, 129])
def test_edges(tiles, n):
    rng = np.random.default_rng(n)
    ops = [_problem(rng, n, m, c) for m, c in ((64, 64), (1, 1), (63, 65), (129, 127), (128, 256), (200, 31))]
    outs, sums = _update(ops, tiles)
    for (a, b), got, s in zip(ops, outs, sums):
        _check(a, b, got, s)


@pytest.mark.parametrize("m, c, n", [
    (40, 40, 4096 + 9),       # 16 columns per packing workgroup, groups read twice
    (40, 40, 1025),           # ... sixteen groups of rows per thread
    (8200, 40, 520),          # 32 columns, eight to sixteen
    (16400, 40, 1100),        # 64 columns, read twice
    (16400, 40, 513),         # 64 columns, sixteen
])
def test_forms_of_the_packing_launch(m, c, n):
    rng = np.random.default_rng(m + n)
    a, b = _problem(rng, n, m, c)
    outs, sums = _update([(a, b)], -1)
    _check(a, b, outs[0], sums[0])


@pytest.mark.parametrize("tiles", [0, 1, 2])
def test_columns_of_any_magnitude(tiles):
    # every column has its own scale, from the smallest normal numbers to large ones, and a column of zeros
    rng = np.random.default_rng(5)
    a, b = _problem(rng, 100, 150, 70, scale_a=lambda m: np.random.default_rng(6).integers(-120, 110, m))
    a[:, 17] = 0.0
    outs, sums = _update([(a, b)], tiles)
    _check(a, b, outs[0], sums[0])
    assert (outs[0][17] == 0).all()


def test_small_elements_beside_large_ones():
    # an element down to 2^-28 of its column's largest keeps its 22 bits
    rng = np.random.default_rng(7)
    a, b = _problem(rng, 96, 80, 80)
    a[0] = 2.0 ** 28
    b[0] = 0.0
    outs, sums = _update([(a, b)], 0)
    ref, mags = a[1:].astype(np.float64).T @ b[1:], np.abs(a[1:]).astype(np.float64).T @ b[1:]
    assert (np.abs(outs[0] - ref) <= (2.0 ** -20 + 15 * 2.0 ** -24) * mags + 96 * 2.0 ** -51 * 2.0 ** 29).all()


@pytest.mark.parametrize("tiles", [0, 1, 2])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_non_finite_operands(tiles, bad):
    # an infinite or undefined operand spoils its row (or column) of the result, and nothing else
    rng = np.random.default_rng(8)
    a, b = _problem(rng, 90, 130, 140)
    a[40, 70] = bad
    outs, _ = _update([(a, b)], tiles, bias=False)
    got = outs[0]
    rest = np.arange(130) != 70
    ref, mags = a.astype(np.float64)[:, rest].T @ b, np.abs(a[:, rest]).astype(np.float64).T @ b
    assert (np.abs(got[rest] - ref) <= (2.0 ** -21 + 15 * 2.0 ** -24) * mags).all()
    assert np.isnan(got[70]).all() if np.isnan(bad) else (got[70] == np.where(b[40] > 0, bad, got[70])).all()


def test_accumulates_onto_parameters_in_whole_lines_and_beyond():
    # 256 x 128: rows of whole cache lines, updated past the L2s; 256 x 100: not
    rng = np.random.default_rng(9)
    ops = [_problem(rng, 80, 256, c) for c in (128, 100)]
    for tiles in (0, 1, 2):
        outs, _ = _update(ops, tiles, c0=3.0)
        for (a, b), got in zip(ops, outs):
            ref = 3.0 + a.astype(np.float64).T @ b.astype(np.float64)
            assert np.abs(got - ref).max() <= 2e-6 * np.abs(ref).max()


def test_arguments():
    x = torch.zeros(64, 64, device="cuda")
    pr = [B.gemm_problem(x, 64, x, 64, torch.zeros_like(x), 64, 64, 64, 64, epi=4, alpha=1.0, beta=1.0)]
    need = B.mavg_gemm_grouped_packed_bytes(pr)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    with pytest.raises(Exception):
        B.mavg_gemm_grouped_packed(pr, -1, ws, workspace_bytes=need - 1)
    with pytest.raises(Exception):
        B.mavg_gemm_grouped_packed(pr, 3, ws)
    pr[0].epi = 0
    with pytest.raises(Exception):
        B.mavg_gemm_grouped_packed(pr, -1, ws)
