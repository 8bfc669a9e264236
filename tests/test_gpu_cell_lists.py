"""The update of short vectors cell by cell, each cell the sum of the coordinates that its list names."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc
from paper_1903_04488_amd.pipeline import DenseStatePath, GraphedStep, HotPath

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _lists(p, d):
    r, c = p.r, p.c
    lists = torch.empty(4 * r * (c + 1 + d), dtype=torch.uint8, device=DEV)
    cs.cs_cell_lists_build(p, d, lists)
    return lists


def _vectors(d, W):
    """small whole numbers: every sum is exact in binary32"""
    base = torch.randint(-8, 9, (d,), generator=torch.Generator().manual_seed(d)).float()
    by = [1 + w % 7 if w % 2 else -(1 + w % 5) for w in range(W)]
    return base, by, [(base * b).to(DEV) for b in by]


# 8, 16, 32 and 64 lanes of a cell, one, two and four wavefronts that share the groups of workers, cells without a
# coordinate and with thousands, more coordinates than lanes take at once, odd sizes
SHAPES = [(1, 1, 1, 1), (3, 7, 5, 3), (5, 33, 1, 9), (7, 40, 784, 4), (5, 33, 2000, 8), (3, 32, 20_011, 17), (15, 64, 1300, 33),
          (5, 1000, 5003, 25), (9, 4096, 50_001, 2), (3, 20_011, 100_003, 31), (5, 8192, 30_000, 256), (1, 2, 4099, 1)]


@pytest.mark.parametrize("r,c,d,W", SHAPES)
def test_tables_merge_and_momentum(r, c, d, W):
    p = cs.cs_params_init(r, c, 190304488, d)
    base, by, gs = _vectors(d, W)
    table = np.asarray(orc.SketchOracle(r, c, 190304488).sketch(base.numpy().astype(np.float64), scale=1.0),
                       dtype=np.float32).reshape(r, c)
    lists = _lists(p, d)
    T = torch.full((cs.cs_bundle_floats(p, W),), float("nan"), device=DEV)
    S_t = torch.full((r, c), float("nan"), device=DEV)
    S_u, S_v = torch.ones(r, c, device=DEV), torch.full((r, c), 2.0, device=DEV)
    cs.cs_bundle_sketch_lists(p, T, gs, lists, 2.0, S_t, 0.5, S_u, S_v, 0.5)
    bundle = T.cpu().numpy().reshape(-1, r, c, 8)
    for w in range(8 * bundle.shape[0]):
        want = table * np.float32(2 * by[w]) if w < W else np.zeros_like(table)
        np.testing.assert_array_equal(bundle[w // 8, :, :, w % 8], want, err_msg=f"slot {w}")
    total = table * np.float32(sum(by))
    np.testing.assert_array_equal(S_t.cpu().numpy(), total)
    np.testing.assert_array_equal(S_u.cpu().numpy(), total + np.float32(0.5))
    np.testing.assert_array_equal(S_v.cpu().numpy(), total + np.float32(2.5))
    only = torch.full((r, c), float("nan"), device=DEV)
    cs.cs_bundle_sketch_lists(p, None, gs, lists, 1.0, only, 1.0)
    np.testing.assert_array_equal(only.cpu().numpy(), total)
    T.fill_(float("nan"))
    cs.cs_bundle_sketch_lists(p, T, gs, lists, 2.0)
    np.testing.assert_array_equal(T.cpu().numpy().reshape(bundle.shape), bundle)


# cells with fewer coordinates than lanes and with more, of one and of several wavefronts; with 16 workers four lanes a coordinate
@pytest.mark.parametrize("r,c,d", [(5, 40, 784), (3, 33, 2001), (3, 7, 5), (5, 1000, 5003), (5, 1000, 3001), (3, 1311, 656), (3, 32, 20_011),
                                   (9, 4096, 50_001)])
@pytest.mark.parametrize("W", [2, 4, 7, 8, 9, 17, 256])
def test_folded_workers_are_summed_before_a_cell_is(r, c, d, W):
    """without worker tables: a cell is off by roundings of the workers' mean, also where the workers all but cancel"""
    gen = torch.Generator().manual_seed(W + d)
    p = cs.cs_params_init(r, c, 190304488, d)
    gs = [1e4 * torch.randn(d, generator=gen) for _ in range(W - 1)]
    gs.append(-sum(g.double() for g in gs).float() + torch.randn(d, generator=gen))
    gs = [g.to(DEV) for g in gs]
    got = torch.full((3, r, c), 0.5, device=DEV)
    cs.cs_bundle_sketch_lists(p, None, gs, _lists(p, d), 1.0, got[0], 1.0 / W, got[1], got[2], 0.5)
    assert torch.equal(got[1], got[0] + 0.25) and torch.equal(got[2], got[1] + 0.5)
    exact = sum(g.double() for g in gs) / W
    bucket, sign = torch.empty(r, d, dtype=torch.int32, device=DEV), torch.empty(r, d, dtype=torch.int8, device=DEV)
    cs.cs_hash_debug_range(p, 0, d, bucket, sign)
    for j in range(r):
        cell = lambda x: torch.zeros(c, dtype=torch.float64, device=DEV).index_add_(0, bucket[j].long(), x)   # noqa: B023, E731
        # n values rounded once and n - 1 additions, each off by half an ulp of at most the sum of magnitudes; twice that
        bound = 2.0 ** -23 * cell(torch.ones_like(exact)) * cell(exact.abs())
        assert ((got[0][j].double() - cell(exact * sign[j])).abs() <= bound).all()


def test_values_that_are_not_finite_stay_in_their_cells():
    r, c, d = 3, 64, 3001
    p = cs.cs_params_init(r, c, 5, d)
    g = torch.zeros(d, device=DEV)
    g[17], g[2000] = float("nan"), float("inf")
    bucket, sign = torch.empty(r, d, dtype=torch.int32, device=DEV), torch.empty(r, d, dtype=torch.int8, device=DEV)
    cs.cs_hash_debug_range(p, 0, d, bucket, sign)
    S = torch.zeros(r, c, device=DEV)
    cs.cs_bundle_sketch_lists(p, None, [g], _lists(p, d), 1.0, S, 1.0)
    for j in range(r):
        nan, inf = int(bucket[j, 17]), int(bucket[j, 2000])
        assert torch.isnan(S[j, nan]) and (nan == inf or S[j, inf] == float("inf") * int(sign[j, 2000]))
        rest = [b for b in range(c) if b not in (nan, inf)]
        assert not S[j, rest].any()


def test_arguments():
    p, d = cs.cs_params_init(5, 33, 1, 500), 500
    lists, g = _lists(p, d), [torch.zeros(d, device=DEV)]
    S = torch.zeros(5, 33, device=DEV)
    with pytest.raises(cs.CsError):
        cs.cs_bundle_sketch_lists(p, None, g, lists)                     # nothing to write
    with pytest.raises(cs.CsError):
        cs.cs_bundle_sketch_lists(p, None, g * 257, lists, S_t=S)
    with pytest.raises(cs.CsError):
        cs.cs_bundle_sketch_lists(p, None, g, lists[:-4].contiguous(), S_t=S)
    with pytest.raises(cs.CsError):
        cs.cs_bundle_sketch_lists(p, None, g, lists, S_t=S, S_u=S)       # one table of the two


def test_more_columns_than_a_launch_takes():
    """8 cells a workgroup of 256 threads: 2^27 columns and more would be a launch of 2^32 threads"""
    r, c, d, W = 1, (1 << 27) + 3, 2001, 25
    p = cs.cs_params_init(r, c, 190304488, d)
    _, _, gs = _vectors(d, W)
    got, want = (torch.zeros(cs.cs_bundle_floats(p, W), device=DEV) for _ in range(2))
    got.fill_(float("nan"))
    cs.cs_bundle_sketch_lists(p, got, gs, _lists(p, d))
    cs.cs_sketch_accumulate_bundle(p, want, gs)
    assert torch.equal(got, want)


@pytest.mark.parametrize("kind", ["step", "fold", "fold-many", "dense", "graph"])
def test_a_path_of_short_vectors_goes_by_its_lists(kind):
    """the same state and selection as a path that is given none, whose atomic additions come in any order: whole numbers, powers
    of two of workers and halves of momentum keep every sum of the three steps a multiple of 2^-8 below 2^15, so that none is
    rounded (with normal values a cell of 500 coordinates and a large one was off by 2e-4 in one run of many)"""
    r, c, d, W, k = 5, 40, 784, 32 if kind == "fold-many" else 4, 2
    d = 20_003 if kind == "fold-many" else d
    gs = [torch.randint(-4, 5, (d,), generator=torch.Generator().manual_seed(w)).float().to(DEV) for w in range(W)]
    for g in gs:
        g[5], g[300] = 400.0, -500.0
    paths = []
    for lists in (True, False):
        cls = DenseStatePath if kind == "dense" else HotPath
        fold = {"fold_workers": True} if kind.startswith("fold") else {}
        path = cls(d, W, r, c, k, 3, rho=0.5, **fold)
        assert path._cell_lists and path._index is not None
        if not lists:
            path._index = None
        step = GraphedStep(path, gs).replay if kind == "graph" and lists else lambda: path.step(gs)   # noqa: B023
        for _ in range(3):
            step()
        paths.append(path)
    a, b = paths
    assert torch.equal(a.S_t, b.S_t) and float(a.S_t.abs().max()) < 2.0 ** 15
    assert a.idx.tolist() == b.idx.tolist() and torch.equal(a.x, b.x)
    if a.S_v is not None:
        assert torch.equal(a.S_v, b.S_v) and torch.equal(a.S_u, b.S_u) and float(a.S_v.abs().max()) < 2.0 ** 15
    # another sketch: not by these lists
    p2 = cs.cs_params_init(r, c, 4, d)
    for path in paths:
        path.params = p2
        path.accumulate(gs if kind != "dense" else path.v_w)
        if not kind.startswith("fold"):
            path.merge()
    assert torch.equal(a.S_t, b.S_t)
