"""cs_bundle_sketch: the update by way of running sums that are gathered by cell, at the edges of its tiles."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc
from paper_1903_04488_amd.pipeline import HotPath
from parity_util import assert_cells_close, sketch_in_slices

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
G = cs.CS_BUNDLE_GROUP
P = (1 << 61) - 1


def _index(p, d):
    index = torch.empty(cs.cs_update_index_bytes(p, 1, d), dtype=torch.uint8, device=DEV)
    cs.cs_update_index_build(p, d, index)
    return index


def _workspace(p, W, d, groups=None):
    """for so many groups of 8 workers at a time"""
    n = cs.cs_update_workspace_bytes(p, W, d)
    return torch.empty(n if groups is None else n // -(-W // G) * groups, dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("W,at_once", [(1, 1), (2, 1), (3, 1), (5, 1), (8, 1), (9, 1), (16, 2), (20, 2), (20, 3)])
@pytest.mark.parametrize("r,c,d", [(5, 64, 4097), (5, 1 << 12, 255_999), (15, 1 << 12, 300_001),
                                   (5, 1 << 15, 1_048_579), (5, 1 << 15, 3_200_003)])
def test_tables_merge_and_momentum(W, at_once, r, c, d):
    if r * d * W > 90_000_000:
        pytest.skip("the long vectors are for three and four sums and the long runs of a walker")
    p = cs.cs_params_init(r, c, 31, d)
    sk = orc.SketchOracle(r, c, 31)
    rng = np.random.default_rng(d + W)
    gs = [(rng.standard_normal(d) * 0.01).astype(np.float32) for _ in range(W)]
    dev = [torch.from_numpy(g).to(DEV) for g in gs]
    index, ws = _index(p, d), _workspace(p, W, d, at_once)
    f32 = dict(dtype=torch.float32, device=DEV)
    T = torch.full((cs.cs_bundle_floats(p, W),), float("nan"), **f32)    # written whole, never read
    ws.view(torch.float32).fill_(float("nan"))
    S_t, S_u, S_v = torch.empty(r, c, **f32), torch.randn(r, c, **f32), torch.randn(r, c, **f32)
    u0, v0 = S_u.double().cpu().numpy(), S_v.double().cpu().numpy()
    cs.cs_bundle_sketch(p, T, dev, index, ws, scale=0.5, S_t=S_t, alpha=0.25, S_u=S_u, S_v=S_v, rho=0.75)
    got = T.cpu().numpy().reshape(-1, r, c, G)
    refs = [sketch_in_slices(sk, g, 0.5) for g in gs]
    for w in range(W):
        assert_cells_close(got[w // G, :, :, w % G], refs[w], terms_per_cell=d / c, what=f"worker {w}")
    for w in range(W, got.shape[0] * G):
        assert not got[w // G, :, :, w % G].any()
    # what follows is computed from the tables: merged in binary64 and rounded once, then three roundings more
    merged = 0.25 * np.sum([got[w // G, :, :, w % G].astype(np.float64) for w in range(W)], axis=0)
    u = 0.75 * u0 + merged
    bound = 4 * 2.0 ** -24 * (np.abs(merged) + np.abs(u0) + np.abs(v0))
    for table, want in ((S_t, merged), (S_u, u), (S_v, v0 + u)):
        assert (np.abs(table.cpu().numpy() - want) <= bound).all()
    again = torch.empty_like(T)
    cs.cs_bundle_sketch(p, again, dev, index, ws, scale=0.5)
    torch.testing.assert_close(again, T, rtol=0, atol=0)                 # one order of additions
    if W <= G:
        only = torch.empty_like(S_t)
        cs.cs_bundle_sketch(p, None, dev, index, ws, scale=0.5, S_t=only, alpha=0.25)
        torch.testing.assert_close(only, S_t, rtol=0, atol=0)


# cells of one and two residues up to 51 000 (a narrow table and a long vector); 15 to 33 on both sides of the sort by one
# thread; 1024 cells and more a workgroup of the other one
@pytest.mark.parametrize("r,c,d", [(5, 64, 4097), (5, 64, 100_000), (5, 64, 1_000_000), (5, 64, 20_000_000),
                                   (5, 256, 300_000), (15, 1 << 12, 300_001), (3, 1 << 20, 20_000_000)])
def test_index(r, c, d):
    p = cs.cs_params_init(r, c, 190304488, d)
    words = r * (c + 1) + sum(p.visit[j].gmax for j in range(r))
    index = torch.full((words,), -1, dtype=torch.int32, device=DEV)
    cs.cs_update_index_build(p, d, index.view(torch.uint8))
    got, at, deepest = index.cpu().numpy(), 0, 0
    for j in range(r):
        n = p.visit[j].gmax
        bucket, sign = torch.empty(r * n, dtype=torch.int32, device=DEV), torch.empty(r * n, dtype=torch.int8, device=DEV)
        cs.cs_hash_debug_range(p, 0, n, bucket, sign)
        cell = bucket.view(r, n)[j].cpu().numpy()
        order = np.argsort(cell, kind="stable")          # by cell, ascending within one
        start = np.searchsorted(cell[order], np.arange(c + 1))
        np.testing.assert_array_equal(got[at:at + c + 1], start)
        np.testing.assert_array_equal(got[at + c + 1:at + c + 1 + n], order)
        at += c + 1 + n
        deepest = max(deepest, np.diff(start).max())
    assert at == words and (d != 20_000_000 or c != 64 or deepest > 50_000)


def test_narrow_table():
    """thousands of sums in a cell"""
    r, c, d, W = 5, 64, 3_000_000, 2
    p = cs.cs_params_init(r, c, 190304488, d)
    gs = [torch.randn(d, generator=torch.Generator().manual_seed(w)).to(DEV) for w in range(W)]
    words = r * (c + 1) + sum(p.visit[j].gmax for j in range(r))
    index = torch.empty(4 * words, dtype=torch.uint8, device=DEV)
    cs.cs_update_index_build(p, d, index)
    T = torch.empty(cs.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV)
    cs.cs_bundle_sketch(p, T, gs, index, _workspace(p, W, d))
    for w in range(W):
        ref = sketch_in_slices(orc.SketchOracle(r, c, 190304488), gs[w].cpu().numpy(), 1.0)
        assert_cells_close(T.view(r, c, G)[:, :, w].cpu().numpy(), ref, terms_per_cell=d / c)


@pytest.mark.parametrize("W", [1, 2, 3, 8])
@pytest.mark.parametrize("r,c,d", [(5, 1 << 12, 200_003), (3, 1 << 13, 400_003)])
@pytest.mark.parametrize("below", [1, 0, -(1 << 28), 1 << 28])
def test_hashes_at_the_thresholds(W, r, c, d, below):
    """The bucket hash of a coordinate, and the sign hash of another, moved on by a visit to `below` short of p; a NaN
    and infinities reach the r cells of their coordinates and no others."""
    p = cs.cs_params_init(r, c, 43, d)
    sk = orc.SketchOracle(r, c, 43)
    g = (np.random.default_rng(W).standard_normal(d) * 0.01).astype(np.float32)
    for j in range(r):
        plan = p.visit[j]
        k = plan.K // 2
        s = sum(plan.gaps()[:k])
        for i, own, consts in ((5, p.a[j], (p.b, sk.b)), (9, p.as_[j], (p.bs, sk.bs))):
            for table in consts:                     # the free term puts that hash there
                table[j] = (P - own * s - below - own * i) % P
            g[i + s] = 1.0 + i
    g[[17, d - 1]], g[100] = np.inf, np.nan
    with np.errstate(invalid="ignore"):
        ref = sk.sketch(g)
    gs = [torch.zeros(d, dtype=torch.float32, device=DEV)] * (W - 1) + [torch.from_numpy(g).to(DEV)]
    T = torch.empty(cs.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV)
    cs.cs_bundle_sketch(p, T, gs, _index(p, d), _workspace(p, W, d))
    got = T.view(r, c, G)[:, :, W - 1].cpu().numpy()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    np.testing.assert_array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(ref), ref, 0))
    fin = np.isfinite(ref)
    assert fin.sum() >= ref.size - 3 * r
    assert_cells_close(np.where(fin, got, 0), np.where(fin, ref, 0), terms_per_cell=d / c)


def test_what_is_refused():
    r, c, d, W = 5, 1 << 12, 200_003, 3
    p = cs.cs_params_init(r, c, 11, d)
    g = [torch.zeros(d, dtype=torch.float32, device=DEV)] * W
    T = torch.empty(cs.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV)
    index, ws = _index(p, d), _workspace(p, W, d)
    short = dict(dtype=torch.uint8, device=DEV)
    for bad in (dict(index=index[:-4]), dict(workspace=ws[:1024]), dict(workspace=torch.empty(ws.numel() + 4, **short)[4:]),
                dict(T=None), dict(S_u=torch.zeros(r, c, device=DEV))):
        with pytest.raises(cs.CsError):
            cs.cs_bundle_sketch(p, **{"T": T, "g_w": g, "index": index, "workspace": ws, **bad})
    # lists that do not keep a coordinate within its sums have no index: the visits' values have no place
    forged = cs.CsParams.from_buffer_copy(p)
    ctypes.memset(ctypes.byref(forged.visit[1]), 0, ctypes.sizeof(forged.visit[1]))
    v = forged.visit[1]
    v.K, v.ncell, v.cover, v.gmax, v.cost, v.cost_walk = 3, 2, d, d - 60_022, 1, 2
    v.gap[0], v.gap[3], v.code[0] = 30_011, d - 60_022, 0b110000
    assert cs.cs_update_index_bytes(forged, W, d) == 0 and cs.cs_update_workspace_bytes(forged, W, d) == 0
    with pytest.raises(cs.CsError):
        cs.cs_bundle_sketch(forged, T, g, index, ws)
    for other in ((7, 40, 784), (3, 5001, 400_003), (5, 1 << 12, 1000)):
        p = cs.cs_params_init(other[0], other[1], 1, other[2])
        assert cs.cs_update_index_bytes(p, 1, other[2]) == 0
        with pytest.raises(cs.CsError):
            cs.cs_bundle_sketch(p, torch.empty(cs.cs_bundle_floats(p, 1), dtype=torch.float32, device=DEV),
                                [torch.zeros(other[2], device=DEV)], index, ws)


@pytest.mark.parametrize("fold", [False, True])
def test_a_path_given_another_sketch_sketches_with_that_one(fold):
    """its index is of the sketch that it was made with; the sums are those of the sketch that it has now"""
    r, c, d, W = 5, 1 << 12, 400_003, 2
    if fold:                                         # (a single vector has an index from r d = 10 million on)
        c, d = 1 << 14, 2_600_003
    gs = [torch.randn(d, generator=torch.Generator().manual_seed(w)).to(DEV) for w in range(W)]
    path = HotPath(d, W, r, c, 50, 190304488, rho=0.9, fold_workers=fold)
    assert path._index is not None
    path.step(gs)
    path.params = cs.cs_params_init(r, c, 3, d)
    path.S_u.zero_(), path.S_v.zero_()
    path.step(gs)
    want = sketch_in_slices(orc.SketchOracle(r, c, 3), ((gs[0].double() + gs[1].double()) / 2).float().cpu().numpy(), 1.0)
    assert_cells_close(path.S_t.cpu().numpy(), want, terms_per_cell=d / c)
