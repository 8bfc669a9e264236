"""The update with a wavefront per vector (2 to 8 vectors of 1.2 million coordinates and more, along visit lists of either
kind): vectors of small whole numbers, whose sums are exact, against the same call with the lists switched off, bit for
bit, as requests, as running sums, added up over the workers, and along a list that leads out of the cells it keeps."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _lists(p):
    return p.visit if p.c_pow2 else p.anyc


def _plain(p):
    q = cs.CsParams.from_buffer_copy(p)
    q.flags |= B.CS_FLAG_NO_VISIT_LIST
    return q


def _forged(p, d):
    """lists of about 40 visits whose offsets have nothing to do with the hashes"""
    q = cs.CsParams.from_buffer_copy(p)
    for j in range(q.r):
        v, gaps = _lists(q)[j], [d // 41 + 3 * j, d // 41 + 1001, d // 43 + 7]
        order, left = [], d
        while left > max(gaps):
            order.append(len(order) % 3)
            left -= gaps[order[-1]]
        v.K, v.cover, v.gmax, v.cost = len(order) + 1, d, max(gaps), 1
        if q.c_pow2:
            v.ncell, v.cost_walk = 2 + j % 3, 2
            for t, g in enumerate(gaps + [left]):
                v.gap[t] = g
            for t in range(len(v.code)):
                v.code[t] = 0
            for k, t in enumerate(order + [3]):
                v.code[k // 16] |= t << 2 * (k % 16)
        else:
            v.omega, v.cost_direct = 1 + j % 2, 2
            for k, g in enumerate([gaps[t] for t in order] + [left]):
                v.gap[k] = g
    return q


# both kinds of columns; the shortest vectors of the rule and ones that end within a wavefront's load
@pytest.mark.parametrize("r,c,d", [(5, 1 << 13, 1_200_001), (3, 1 << 15, 3_000_002), (15, 1 << 12, 1_300_003),
                                   (5, 20_011, 1_900_003), (3, 4_999, 1_200_000)])
@pytest.mark.parametrize("W", [2, 3, 4, 5, 8])
def test_tables_and_running_sums(r, c, d, W):
    p = cs.cs_params_init(r, c, 190304488, d)
    lists = _lists(p)
    assert all(lists[j].K > 0 for j in range(r))
    gen = torch.Generator(device=DEV).manual_seed(W)
    g = [torch.randint(-8, 9, (d,), device=DEV, generator=gen).float() for _ in range(W)]
    n = cs.cs_bundle_floats(p, W)
    want = torch.zeros(n, device=DEV)
    cs.cs_sketch_accumulate_bundle(_plain(p), want, g, i0=5, scale=0.5)
    for params in (p, _forged(p, d)):
        got = torch.zeros(n, device=DEV)
        cs.cs_sketch_accumulate_bundle(params, got, g, i0=5, scale=0.5)
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    tables = want.view(r, c, 8)
    S = torch.zeros(r, c, device=DEV)
    cs.cs_sketch_accumulate_sum(p, S, g, i0=5, scale=0.5)
    np.testing.assert_array_equal(S.cpu().numpy(), tables.sum(2).cpu().numpy())
    need = cs.cs_update_workspace_bytes(p, W, d)
    assert (need > 0) == bool(p.c_pow2)
    if need:
        index = torch.empty(4 * (r * (c + 1) + sum(p.visit[j].gmax for j in range(r))), dtype=torch.uint8, device=DEV)
        cs.cs_update_index_build(p, d, index)
        ws = torch.full((need // 4,), float("nan"), device=DEV).view(torch.uint8)
        T, S_t = torch.full((n,), float("nan"), device=DEV), torch.full((r, c), float("nan"), device=DEV)
        cs.cs_bundle_sketch(p, T, g, index, ws, scale=0.5, S_t=S_t)
        want.zero_()
        cs.cs_sketch_accumulate_bundle(_plain(p), want, g, scale=0.5)
        np.testing.assert_array_equal(T.cpu().numpy(), want.cpu().numpy())
        np.testing.assert_array_equal(S_t.cpu().numpy(), want.view(r, c, 8).sum(2).cpu().numpy())
