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
