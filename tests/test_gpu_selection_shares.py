"""Selections that end early and lists that several workgroups write: candidate counts around what one workgroup takes, with
the entry that decides alone in its bin, in a bin that is wanted whole, among equals, and among zeros."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _want(est, k):
    key = est.view(np.uint32) & np.uint32(0x7FFFFFFF)
    order = np.lexsort((np.arange(len(est)), -key.astype(np.int64)))
    return np.sort(order[:k])


def _select(est, k, kept):
    d = len(est)
    ws = torch.empty(cs.cs_topk_workspace_bytes(d, k), dtype=torch.uint8, device=DEV)
    idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
    val = torch.zeros(k, device=DEV)
    cs.cs_topk_workspace_clear(ws)
    dev = torch.from_numpy(est).to(DEV)
    for _ in range(2 if kept else 1):                  # (the workspace is left clear)
        if kept:
            bins = (est.view(np.uint32) & np.uint32(0x7FFFFFFF)) >> np.uint32(20)
            hist = torch.from_numpy(np.bincount(bins, minlength=2048).astype(np.int64)).to(DEV)
            cs.cs_heavy_hitters_topk_kept(dev, k, idx, val, ws, hist)
        else:
            cs.cs_heavy_hitters_topk(dev, k, idx, val, ws)
        want = _want(est, k)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        np.testing.assert_array_equal(val.cpu().numpy(), est[want])


# entries of the deciding bin and above: less and more than a workgroup's share, the most that is shared in LDS, and beyond
@pytest.mark.parametrize("n", [1, 1024, 1025, 2048, 2049, 4097, 16_385, 32_767, 32_768, 32_769])
@pytest.mark.parametrize("kind", ["spread", "whole bin", "equal", "half equal"])
def test_lists(n, kind):
    d = 1 << 20
    rng = np.random.default_rng(n)
    est = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    at = rng.choice(d, n, replace=False)
    big = rng.uniform(1.0, 1.125, n).astype(np.float32)            # one bin of the first histogram
    k = max(1, n // 3)
    if kind == "whole bin":
        k = n
    elif kind == "equal":
        big[:] = 1.0625
    elif kind == "half equal":
        big[: (n + 1) // 2] = 1.0625
    est[at] = big * rng.choice([-1.0, 1.0], n).astype(np.float32)
    _select(est, k, kept=True)


@pytest.mark.parametrize("d", [1, 1000, 2049, 32_768, 300_000])
@pytest.mark.parametrize("nonzero", [0, 1, 100])
def test_among_zeros(d, nonzero):
    """theta is 0 where more are wanted than are not zero; those of the lowest indices are taken"""
    rng = np.random.default_rng(d)
    est = np.zeros(d, dtype=np.float32)
    n = min(nonzero, d)
    est[rng.choice(d, n, replace=False)] = rng.uniform(0.1, 1.0, n).astype(np.float32)
    for k in {max(1, n // 2), max(1, n), min(d, n + 5), min(d, 700)}:
        _select(est, k, kept=False)
