"""The query along visit lists (column counts that are no powers of two) tells a coordinate's cell and sign by
comparing the top 32 bits of its hash with a threshold of the visit; without scratch the same query computes every
hash.  The two have to agree bit for bit, and the counts by magnitude with the estimates."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc
from parity_util import estimate_in_slices

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
P = (1 << 61) - 1


def _scratch(n):
    return torch.empty(n, dtype=torch.uint8, device=DEV) if n else None


# lists with one and two cells per wrap (the third and the last case, there in the last row of 3 and in rows
# before the last of 15); the smallest length served and odd ends
@pytest.mark.parametrize("r,c,d,seed", [(5, 30011, 3 << 19, 47), (3, 50021, 2_200_001, 31), (3, 9001, 2_100_003, 47),
                                        (15, 60000, 1_600_003, 190304488)])
@pytest.mark.parametrize("below", [None, 1, 0, 1 << 28])
@pytest.mark.parametrize("sign", [False, True])
def test_query_with_lists_is_the_query_by_hashes(r, c, d, seed, below, sign):
    p = cs.cs_params_init(r, c, seed, d)
    assert cs.cs_estimate_workspace_bytes(p, d) == 0 and cs.cs_estimate_scratch_bytes(p, d) == 4 * r * d
    i0 = 3
    if below is not None:                            # residue 5 of a visit `below` short of its wrap
        j = r - 1
        k = p.anyc[j].K // 2
        a, b = (p.as_[j], p.bs[j]) if sign else (p.a[j], p.b[j])
        s = int(sum(p.anyc[j].gaps()[:k]))
        i0 = ((P - a * s % P - below - b) * pow(a, -1, P) - 5) % P
        if i0 > P - d:                               # (not reachable with a global index)
            pytest.skip("index base beyond the range of the entry point")
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(d)).to(DEV)
    S[0, 7], S[-1, 11], S[1, 13] = float("inf"), float("nan"), 0.0
    want, want_n = torch.empty(d, device=DEV), torch.full((2048,), 9, dtype=torch.int64, device=DEV)
    cs.cs_sketch_estimate(p, S, want, i0, None, want_n)
    for hist in (None, torch.full((2048,), 9, dtype=torch.int64, device=DEV)):
        got = torch.full((d,), 77.0, device=DEV)
        cs.cs_sketch_estimate(p, S, got, i0, _scratch(4 * r * d), hist)
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    assert torch.equal(hist, want_n)
    # too little scratch, or scratch that floats cannot lie in, is scratch unused
    buf = _scratch(4 * r * d + 1)
    for ws in (buf[:4 * r * d - 1], buf[1:]):
        got = torch.full((d,), 77.0, device=DEV)
        cs.cs_sketch_estimate(p, S, got, i0, ws)
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())


# r d from 200 million on is written in whole lines, wherever the scratch and the result begin; lists with one cell and (the
# second case, 15 rows) with two cells per wrap
@pytest.mark.parametrize("r,c,d", [(5, 180_000, 40_000_001), (15, 250_007, 13_400_003)])
@pytest.mark.parametrize("of_rows,of_est", [(0, 0), (3, 1), (30, 31)])
def test_query_in_whole_lines(r, c, d, of_rows, of_est):
    p = cs.cs_params_init(r, c, 190304488, d)
    n = cs.cs_estimate_scratch_bytes(p, d)
    assert n == 4 * r * d
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(d)).to(DEV)
    want = torch.empty(d, device=DEV)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(3, d + 3, device=DEV), want)
    for hist in (None, torch.full((2048,), 9, dtype=torch.int64, device=DEV)):
        got = torch.full((d + 64,), 77.0, device=DEV)
        est = got[of_est:of_est + d]
        cs.cs_sketch_estimate(p, S, est, 3, _scratch(n + 4 * of_rows)[4 * of_rows:], hist)
        assert torch.equal(est, want)
        assert (got[:of_est] == 77.0).all() and (got[of_est + d:] == 77.0).all()
    bins = (want.abs().view(torch.int32).long() >> 20)
    assert torch.equal(hist, torch.bincount(bins, minlength=2048))


# the same where the lower bits of a hash decide: of a residue of a wavefront's own, and of one of the line behind them that it
# writes as well (lists with one cell and, the second case, with two cells per wrap)
@pytest.mark.parametrize("r,c,d", [(5, 180_000, 40_000_001), (15, 250_007, 13_400_003)])
@pytest.mark.parametrize("row", [0, -1])
@pytest.mark.parametrize("residue", [5, 256 + 21])
@pytest.mark.parametrize("below", [1, 0, 1 << 28])
@pytest.mark.parametrize("sign", [False, True])
def test_query_in_whole_lines_at_the_thresholds(r, c, d, row, residue, below, sign):
    p = cs.cs_params_init(r, c, 190304488, d)
    j = row % r
    k = p.anyc[j].K // 2
    a, b = (p.as_[j], p.bs[j]) if sign else (p.a[j], p.b[j])
    s = int(sum(p.anyc[j].gaps()[:k]))
    i0 = ((P - a * s % P - below - b) * pow(a, -1, P) - residue) % P
    if i0 > P - d:                                   # (not reachable with a global index)
        pytest.skip("index base beyond the range of the entry point")
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(d)).to(DEV)
    want, got = torch.empty(d, device=DEV), torch.empty(d + 1, device=DEV)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(i0, i0 + d, device=DEV), want)
    cs.cs_sketch_estimate(p, S, got[1:], i0, _scratch(cs.cs_estimate_scratch_bytes(p, d)))
    assert torch.equal(got[1:], want)


# strides that differ by a factor of 250 between the rows (one row of 8 wavefronts in 256 segments beside rows of
# 1100 in one), the shortest vector that is walked, and the lengths on both sides of the fused last row
@pytest.mark.parametrize("r,c,d", [(15, 1 << 16, 2_000_000), (5, 1 << 15, 1 << 20), (3, 64, 4096), (1, 1 << 10, 70_001),
                                   (5, 1 << 16, (1 << 24) - 1), (5, 1 << 16, 1 << 24)])
def test_query_by_walks_is_the_query_of_single_coordinates(r, c, d):
    p = cs.cs_params_init(r, c, 190304488, d)
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(d)).to(DEV)
    want = torch.empty(d, device=DEV)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(3, d + 3, device=DEV), want)
    for hist in (None, torch.full((2048,), 9, dtype=torch.int64, device=DEV)):
        got = torch.full((d,), 77.0, device=DEV)
        cs.cs_sketch_estimate(p, S, got, 3, _scratch(cs.cs_estimate_workspace_bytes(p, d)), hist)
        assert torch.equal(got, want)
    bins = (want.abs().view(torch.int32).long() >> 20)
    assert torch.equal(hist, torch.bincount(bins, minlength=2048))


# the median by selection and, where a wavefront meets a NaN, by the sort that the definition has; ties and infinities
@pytest.mark.parametrize("r", [1, 3, 5, 7, 9, 11, 13, 15])
@pytest.mark.parametrize("c", [64, 97])
@pytest.mark.parametrize("nan", [False, True])
def test_medians_of_every_row_count(r, c, nan):
    d = 5003
    p = cs.cs_params_init(r, c, 5, d)
    sk = orc.SketchOracle(r, c, 5)
    rng = np.random.default_rng(r * c)
    T = rng.integers(-3, 4, (r, c)).astype(np.float64)
    T[rng.random((r, c)) < 0.05] = np.inf
    if nan:
        T[rng.random((r, c)) < 0.02] = np.nan
    S = torch.from_numpy(T.astype(np.float32)).to(DEV)
    want = sk.estimate(T, d)
    sparse, est = torch.empty(d, device=DEV), torch.empty(d, device=DEV)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(d, device=DEV), sparse)
    cs.cs_sketch_estimate(p, S, est, 0, _scratch(cs.cs_estimate_workspace_bytes(p, d)))
    np.testing.assert_array_equal(sparse.cpu().numpy(), want)
    np.testing.assert_array_equal(est.cpu().numpy(), want)


def _bits(x):
    return x.view(torch.int32).cpu().numpy()


# every kernel that takes a median: single coordinates hashed (d = 5003), lattice and its median of rows, the walk with the last row
# fused, lists with and without whole lines
@pytest.mark.parametrize("r,c,d", [(1, 64, 5003), (5, 64, 5003), (15, 97, 5003), (3, 1 << 10, 70_001), (15, 1 << 12, 300_001),
                                   (5, 1 << 15, 1 << 24), (5, 30011, 3 << 19), (15, 250_007, 13_400_003)])
@pytest.mark.parametrize("nan", [False, True])
def test_the_sign_of_a_zero_median_is_that_of_the_sort(r, c, d, nan):
    """-0 and +0 are equal and keep the order of the rows, whatever other coordinates of a wavefront hold; the oracle's
    insertion sort in 64 bits has the same zeros"""
    p = cs.cs_params_init(r, c, 7, d)
    rng = np.random.default_rng(r * c)
    T = rng.integers(-1, 2, (r, c)) * (rng.random((r, c)) < 0.5) * np.where(rng.random((r, c)) < 0.5, -1.0, 1.0)
    if nan:
        T[rng.integers(0, r), rng.integers(0, c)] = np.nan
    S = torch.from_numpy(T.astype(np.float32)).to(DEV)
    want = estimate_in_slices(orc.SketchOracle(r, c, 7), T, d)
    number = ~np.isnan(want)
    bits = want.astype(np.float32).view(np.int32)
    assert {0, -(1 << 31)} <= set(bits[number].tolist())
    est, sparse = torch.empty(d, device=DEV), torch.empty(d, device=DEV)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(d, device=DEV), sparse)
    for hist in (None, torch.empty(2048, dtype=torch.int64, device=DEV)):
        cs.cs_sketch_estimate(p, S, est, 0, _scratch(cs.cs_estimate_scratch_bytes(p, d)), hist)
        for got in (est, sparse):
            np.testing.assert_array_equal(torch.isnan(got).cpu().numpy(), ~number)
            np.testing.assert_array_equal(_bits(got)[number], bits[number])
