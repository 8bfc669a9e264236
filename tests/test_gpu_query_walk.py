"""The query of power-of-two column counts follows a stride, tells cell and sign of a coordinate by comparing its
hash with a threshold of the visit and takes cells four at a time; the query of listed coordinates computes every
hash.  The two have to agree bit for bit, and the counts by magnitude with the estimates."""
import pytest
import torch

import paper_1903_04488_amd as cs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
P = (1 << 61) - 1


def _check(p, S, d, i0, of_rows=0, of_est=0):
    r = p.r
    want = torch.empty(d, device=DEV)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(i0, i0 + d, device=DEV), want)
    want_n = torch.bincount((want.view(torch.int32) & 0x7FFFFFFF) >> 20, minlength=2048)
    for hist in (None, torch.full((2048,), 9, dtype=torch.int64, device=DEV)):
        ws = torch.empty(4 * (r * d + of_rows), dtype=torch.uint8, device=DEV)[4 * of_rows:]
        buf = torch.full((d + of_est + 40,), 77.0, device=DEV)
        cs.cs_sketch_estimate(p, S, buf[of_est:of_est + d], i0, ws, hist)
        assert torch.equal(buf[of_est:of_est + d].view(torch.int32), want.view(torch.int32))
        assert bool((buf[:of_est] == 77.0).all()) and bool((buf[of_est + d:] == 77.0).all())
    assert torch.equal(hist, want_n)


def _table(r, c, seed):
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(seed)).to(DEV)
    S[0, 7], S[-1, 11], S[0, c - 1], S[-1, 0] = float("inf"), float("nan"), -float("inf"), -0.0
    return S


# the smallest served, narrow tables (many cells at a row's end), one row, the last row with and without the median,
# below and in whole lines (from r d = 75 million, 120 million with many rows)
SHAPES = [(5, 64, 4096), (7, 64, 100_003), (1, 1 << 12, 300_007), (3, 1 << 15, 1_000_003), (5, 1 << 12, 4_999_999),
          (5, 1 << 17, 5_000_001), (3, 1 << 16, 25_000_003), (7, 1 << 17, 10_714_289), (15, 1 << 16, 8_000_009)]


@pytest.mark.parametrize("r,c,d", SHAPES)
@pytest.mark.parametrize("below", [None, 1, 0])
@pytest.mark.parametrize("sign", [False, True])
def test_query_by_thresholds_is_the_query_by_hashes(r, c, d, below, sign):
    p = cs.cs_params_init(r, c, 190304488 + d, d)
    if cs.cs_estimate_scratch_bytes(p, d) == 0 or p.plan[r - 1].Dw <= 1:
        pytest.skip("no stride for this sketch")
    i0 = 3
    if below is not None:                            # residue 5 of visit 3 `below` short of its wrap
        a, b = (p.as_[r - 1], p.bs[r - 1]) if sign else (p.a[r - 1], p.b[r - 1])
        i0 = ((P - a * 3 * p.plan[r - 1].Dw % P - below - b) * pow(a, -1, P) - 5) % P
        if i0 > P - d:
            pytest.skip("index base beyond the range of the entry point")
    _check(p, _table(r, c, d), d, i0)


@pytest.mark.parametrize("of_rows,of_est", [(3, 1), (30, 31)])
@pytest.mark.parametrize("r,c,d", [(5, 1 << 17, 5_000_001), (3, 1 << 16, 25_000_003), (15, 1 << 16, 8_000_009)])
def test_scratch_and_result_may_begin_anywhere(r, c, d, of_rows, of_est):
    p = cs.cs_params_init(r, c, 47, d)
    _check(p, _table(r, c, d), d, 1, of_rows, of_est)


# strides that lead up and down, by less and by more than a cell a visit
@pytest.mark.parametrize("stride", [1, 12_345, 40_961])
@pytest.mark.parametrize("up", [False, True])
def test_any_stride(stride, up):
    r, c, d = 3, 64, 200_003
    p = cs.cs_params_init(r, c, 11, d)
    for j in range(r):
        s = stride + 1 + j
        if up:                                       # (another stride with its own advances is as good a plan)
            s = max(2, p.plan[j].Dw // 3)
        p.plan[j].Dw, p.plan[j].ADw, p.plan[j].ADws = s, p.a[j] * s % P, p.as_[j] * s % P
    _check(p, _table(r, c, d), d, 5)
