"""The update where the workgroups of a launch are more than the chip holds at a time (at most 32 wavefronts on each of 256
CUs), so that some walk their visits down and some up: vectors of small whole numbers, whose sums are exact, against the
same call with the lists switched off, bit for bit."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _plain(p):
    q = cs.CsParams.from_buffer_copy(p)
    q.flags |= B.CS_FLAG_NO_VISIT_LIST
    return q


# (a wavefront has 256 residues of one vector, 128 of eight, 256 of four)
@pytest.mark.parametrize("r,c,d,W", [(7, 1 << 18, 12_000_001, 8), (7, 1 << 18, 12_000_003, 5), (5, 1 << 20, 22_000_002, 3),
                                     (7, 1 << 20, 20_000_005, 1), (5, 250_007, 7_000_001, 8), (5, 1_000_003, 22_000_001, 1)])
def test_more_workgroups_than_the_chip_holds(r, c, d, W):
    p = cs.cs_params_init(r, c, 190304488, d)
    lists = p.visit if p.c_pow2 else p.anyc
    assert all(lists[j].K > 0 for j in range(r))
    assert sum(lists[j].gmax for j in range(r)) > 32 * 256 * (128 if W > 4 else 256)
    gen = torch.Generator(device=DEV).manual_seed(W)
    g = [torch.randint(-8, 9, (d,), device=DEV, generator=gen).float() for _ in range(W)]
    n = cs.cs_bundle_floats(p, W)
    want, got = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    cs.cs_sketch_accumulate_bundle(_plain(p), want, g, scale=0.5)
    cs.cs_sketch_accumulate_bundle(p, got, g, scale=0.5)
    np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    S = torch.zeros(r, c, device=DEV)
    cs.cs_sketch_accumulate_sum(p, S, g, scale=0.5)
    np.testing.assert_array_equal(S.cpu().numpy(), want.view(r, c, 8).sum(2).cpu().numpy())
    index_bytes = cs.cs_update_index_bytes(p, W, d)
    if index_bytes:
        index = torch.empty(index_bytes, dtype=torch.uint8, device=DEV)
        cs.cs_update_index_build(p, d, index)
        ws = torch.full((cs.cs_update_workspace_bytes(p, W, d) // 4,), float("nan"), device=DEV).view(torch.uint8)
        T = torch.full((n,), float("nan"), device=DEV)
        cs.cs_bundle_sketch(p, T, g, index, ws, scale=0.5)
        np.testing.assert_array_equal(T.cpu().numpy(), want.cpu().numpy())
