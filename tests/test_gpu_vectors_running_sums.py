"""The running sums that a wavefront per vector writes to the workspace of the two-pass update, with two, three and four of them
beside each other in a launch: vectors of small whole numbers, whose sums are exact, against the update with the lists switched off, bit
for bit, on a workspace of NaN."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (15 rows: two launches, of 8 and of 7)
@pytest.mark.parametrize("r,c,d,sums", [(5, 1 << 15, 2_000_003, 4), (5, 1 << 16, 3_300_001, 4), (3, 1 << 16, 4_500_001, 3),
                                        (15, 1 << 14, 2_000_003, 3)])
@pytest.mark.parametrize("W", [2, 3, 4, 7, 8])
def test_gathered_sums(r, c, d, sums, W):
    p = cs.cs_params_init(r, c, 190304488, d)
    of_rows = [p.visit[j].ncell for j in range(r)]
    residues = sum(p.visit[j].gmax for j in range(r))
    assert max(of_rows) == sums and min(of_rows) == 2
    assert r * d >= 25 * residues and residues >= 200_000 and 4 * d * 8 <= 3.4e8
    need = cs.cs_update_workspace_bytes(p, W, d)
    assert need > 0
    plain = cs.CsParams.from_buffer_copy(p)
    plain.flags |= B.CS_FLAG_NO_VISIT_LIST
    gen = torch.Generator(device=DEV).manual_seed(W)
    g = [torch.randint(-8, 9, (d,), device=DEV, generator=gen).float() for _ in range(W)]
    n = cs.cs_bundle_floats(p, W)
    want = torch.zeros(n, device=DEV)
    cs.cs_sketch_accumulate_bundle(plain, want, g, scale=0.5)
    index = torch.empty(4 * (r * (c + 1) + sum(p.visit[j].gmax for j in range(r))), dtype=torch.uint8, device=DEV)
    cs.cs_update_index_build(p, d, index)
    ws = torch.full((need // 4,), float("nan"), device=DEV).view(torch.uint8)
    T, S_t = torch.full((n,), float("nan"), device=DEV), torch.full((r, c), float("nan"), device=DEV)
    cs.cs_bundle_sketch(p, T, g, index, ws, scale=0.5, S_t=S_t)
    np.testing.assert_array_equal(T.cpu().numpy(), want.cpu().numpy())
    np.testing.assert_array_equal(S_t.cpu().numpy(), want.view(r, c, 8).sum(2).cpu().numpy())
