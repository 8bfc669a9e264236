"""Groups of workers of short vectors share a launch: every worker's table, whatever the number of groups.

Vectors are small whole numbers and worker w's is a multiple of the first's, so that every sum is exact in binary32 and
the tables are compared bit for bit."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _vectors(d, W, seed=1):
    base = torch.randint(-8, 9, (d,), generator=torch.Generator().manual_seed(seed)).float()
    by = [1 + w % 7 if w % 2 else -(1 + w % 5) for w in range(W)]
    return base, by, [(base * b).to(DEV) for b in by]


def _oracle(r, c, seed, base):
    table = orc.SketchOracle(r, c, seed).sketch(base.numpy().astype(np.float64), scale=1.0)
    return np.asarray(table, dtype=np.float32).reshape(r, c)


def _assert_bundle(T, table, by, r, c):
    T = T.cpu().numpy().reshape(-1, r, c, 8)
    for w, b in enumerate(by):
        np.testing.assert_array_equal(T[w // 8, :, :, w % 8], table * np.float32(b), err_msg=f"worker {w}")
    for w in range(len(by), 8 * T.shape[0]):
        assert not T[w // 8, :, :, w % 8].any(), f"slot {w} belongs to no worker"


# column counts with lists of three gaps and with gaps one by one; W: a launch of two groups, with a tail of one
# worker, more groups than a launch takes (32 and 8); few and many rows
@pytest.mark.parametrize("r,c,d,W", [
    (3, 256, 40_003, 16), (5, 512, 50_001, 17), (9, 128, 20_011, 25), (3, 64, 8_001, 257), (3, 64, 8_001, 300),
    (5, 1000, 70_003, 9), (3, 701, 66_001, 64), (7, 701, 66_001, 65), (3, 701, 66_001, 140)])
def test_requests_of_several_groups(r, c, d, W):
    p = cs.cs_params_init(r, c, 190304488, d)
    base, by, gs = _vectors(d, W)
    table = _oracle(r, c, 190304488, base)
    T = torch.zeros(cs.cs_bundle_floats(p, W), device=DEV)
    cs.cs_sketch_accumulate_bundle(p, T, gs)
    _assert_bundle(T, table, by, r, c)
    S = torch.zeros(r, c, device=DEV)
    cs.cs_sketch_accumulate_sum(p, S, gs)
    np.testing.assert_array_equal(S.cpu().numpy(), table * np.float32(sum(by)))


# the running sums of all groups, of a few at a time and of one at a time
@pytest.mark.parametrize("r,c,d,W", [(5, 256, 50_001, 9), (3, 1 << 12, 300_007, 31), (9, 128, 30_011, 300)])
@pytest.mark.parametrize("groups", [1, 2, 3, 1000])
def test_running_sums_of_several_groups(r, c, d, W, groups):
    p = cs.cs_params_init(r, c, 190304488, d)
    base, by, gs = _vectors(d, W)
    table = _oracle(r, c, 190304488, base)
    need = cs.cs_update_workspace_bytes(p, W, d)
    assert need > 0
    all_groups = -(-W // 8)
    ws = torch.empty(need // all_groups * min(groups, all_groups), dtype=torch.uint8, device=DEV)
    index = torch.empty(4 * (r * (c + 1) + sum(p.visit[j].gmax for j in range(r))), dtype=torch.uint8, device=DEV)
    cs.cs_update_index_build(p, d, index)
    T = torch.full((cs.cs_bundle_floats(p, W),), float("nan"), device=DEV)
    S_t = torch.full((r, c), float("nan"), device=DEV)
    cs.cs_bundle_sketch(p, T, gs, index, ws, S_t=S_t)
    _assert_bundle(T, table, by, r, c)
    np.testing.assert_array_equal(S_t.cpu().numpy(), table * np.float32(sum(by)))
