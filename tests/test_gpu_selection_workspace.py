"""Selections that share one kept workspace, and what becomes of one whose counters are not clear."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# where the counter lies from which workgroups draw their tasks: behind three histograms of 2048
# 64-bit counts, two 32-bit words and a 64-bit count
TICKET = 3 * 2048 * 8 + 2 * 4 + 8


@pytest.mark.parametrize("with_val", [True, False])
def test_selection_with_a_stale_counter_ends_and_shows_it(with_val):
    """The first task is never drawn, so the workgroups that wait for it give up: indices in range, NaN
    values, and a workspace that serves the next selection."""
    d, k = 200_003, 1000
    est = (np.random.default_rng(1).standard_normal(d)).astype(np.float32)
    dev_est = torch.from_numpy(est).to(DEV)
    # (a call without a histogram clears the workspace first)
    bins = (est.view(np.uint32) & np.uint32(0x7FFFFFFF)) >> np.uint32(20)
    hist = torch.from_numpy(np.bincount(bins, minlength=2048).astype(np.int64)).to(DEV)
    # the fixed part alone, so that est itself is shared out among the workgroups
    ws = torch.zeros(cs.cs_topk_workspace_bytes(1, 1), dtype=torch.uint8, device=DEV)
    cs.cs_topk_workspace_clear(ws)
    idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
    val = torch.zeros(k, dtype=torch.float32, device=DEV) if with_val else None
    ws[TICKET:TICKET + 4].view(torch.int32).fill_(1)
    cs.cs_heavy_hitters_topk_kept(dev_est, k, idx, val, ws, hist)
    np.testing.assert_array_equal(idx.cpu().numpy(), np.arange(k))
    if with_val:
        assert torch.isnan(val).all()
    want = orc.topk_threshold(est, k)
    for _ in range(2):
        cs.cs_heavy_hitters_topk_kept(dev_est, k, idx, val, ws, hist)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        if with_val:
            np.testing.assert_array_equal(val.cpu().numpy(), est[want])


def test_one_kept_workspace_serves_every_kind_of_selection_in_turn():
    """Each leaves the workspace clear for the next: ordinary lists, a list that is too long for one
    workgroup, lists that cannot be built (one stretch of heavy entries, all magnitudes in one bin),
    HEAVYMIX with its list and without, P k candidates, and vectors of one workgroup."""
    d = 3_000_017
    rng = np.random.default_rng(5)
    noise = (rng.standard_normal(d) * 0.01).astype(np.float32)
    stretch = noise.copy()
    stretch[700_000:709_000] = rng.uniform(0.5, 1.0, size=9000).astype(np.float32)
    one_bin = (rng.uniform(1.0, 1.05, size=d) * rng.choice([-1.0, 1.0], size=d)).astype(np.float32)
    ws = torch.full((cs.cs_topk_workspace_bytes(d, 60_000),), 0xA7, dtype=torch.uint8, device=DEV)
    cs.cs_topk_workspace_clear(ws)

    def kept(est, k):
        dev_est = torch.from_numpy(est).to(DEV)
        bins = (est.view(np.uint32) & np.uint32(0x7FFFFFFF)) >> np.uint32(20)
        hist = torch.from_numpy(np.bincount(bins, minlength=2048).astype(np.int64)).to(DEV)
        idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
        val = torch.empty(k, dtype=torch.float32, device=DEV)
        cs.cs_heavy_hitters_topk_kept(dev_est, k, idx, val, ws, hist)
        want = orc.topk_threshold(est, k)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        np.testing.assert_array_equal(val.cpu().numpy().view(np.uint32), est[want].view(np.uint32))

    def heavymix(est, k, l2sq):
        idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
        val = torch.empty(k, dtype=torch.float32, device=DEV)
        n_heavy = torch.full((1,), -1, dtype=torch.int64, device=DEV)
        cs.cs_heavymix_select(torch.from_numpy(est).to(DEV), k, torch.tensor([l2sq], dtype=torch.float64, device=DEV), 9,
                              idx, val, n_heavy, ws)
        want, heavy = orc.heavymix_select(est, k, l2sq, 9)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        assert int(n_heavy.item()) == heavy

    def exact(n, k):
        cand = np.sort(rng.choice(10**8, n, replace=False)).astype(np.int64)
        x = (np.round(rng.standard_normal(n) * 50) / 50).astype(np.float32)      # ties
        idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
        val = torch.empty(k, dtype=torch.float32, device=DEV)
        cs.cs_select_exact_topk(torch.from_numpy(cand).to(DEV), torch.from_numpy(x).to(DEV), k, idx, val, ws)
        np.testing.assert_array_equal(idx.cpu().numpy(), cand[orc.topk_threshold(x, k)])

    for step in (lambda: kept(stretch, 2000), lambda: kept(one_bin, 2000), lambda: heavymix(noise, 3000, 1e-12),
                 lambda: heavymix(noise, 3000, 1e12), lambda: exact(200_000, 3000), lambda: kept(noise, 60_000),
                 lambda: kept(noise[:20_000].copy(), 5), lambda: exact(500, 20)):
        kept(noise, 2000)
        step()
        kept(noise, 2000)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("k", [3_000, 300_000, 400_001])
def test_selection_from_crowded_parts_and_long_segments(offset, k):
    """Parts of the vector with more candidates than a wavefront stages (2048 of 2048, and half of them),
    a list with more than 512 candidates per segment, and equal magnitudes at the k-th place, with and
    without room for the list, and as HEAVYMIX."""
    d = 8_400_005
    rng = np.random.default_rng(k + offset)
    est = (rng.standard_normal(d) * 0.01).astype(np.float32)
    some = rng.choice(d, 500_000, replace=False)
    est[some] = (rng.integers(16, 31, size=some.size) / 16 * rng.choice([-1.0, 1.0], size=some.size)).astype(np.float32)
    est[1_000_001:1_009_000] = 1.5
    est[5_000_000:5_040_000:2] = -1.25
    base = torch.zeros(d + 1, dtype=torch.float32, device=DEV)
    view = base[offset:offset + d]
    view.copy_(torch.from_numpy(est))
    want = orc.topk_threshold(est, k)
    full, bare = cs.cs_topk_workspace_bytes(d, k), cs.cs_topk_workspace_bytes(1, 1)
    assert full > bare + 12 * (2 * k + 4096)
    for nbytes in (full, bare):
        ws = torch.full((nbytes,), 0x3D, dtype=torch.uint8, device=DEV)
        idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
        val = torch.empty(k, dtype=torch.float32, device=DEV)
        cs.cs_heavy_hitters_topk(view, k, idx, val, ws)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        np.testing.assert_array_equal(val.cpu().numpy(), est[want])
        n_heavy = torch.full((1,), -1, dtype=torch.int64, device=DEV)
        l2sq = float(k) * 1.2 ** 2                                  # heavy: magnitudes of 1.25 and more
        cs.cs_heavymix_select(view, k, torch.tensor([l2sq], dtype=torch.float64, device=DEV), 5, idx, val, n_heavy, ws)
        mix, heavy = orc.heavymix_select(est, k, l2sq, 5)
        np.testing.assert_array_equal(idx.cpu().numpy(), mix)
        assert int(n_heavy.item()) == heavy
