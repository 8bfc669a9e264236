"""The update along visit lists in runs of 16, whose launches send two neighbouring cells of a bundle as one request or every
cell by itself (by the running sums, the workers and the columns): vectors of small whole numbers, whose sums are exact, against
the same call with the lists switched off, bit for bit."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# two, three and four sums on either side of 2^17 columns, at 64 coordinates a column (two sums) and more
@pytest.mark.parametrize("r,c,d,seed,sums", [(3, 1 << 17, 3_300_002, 19, 2), (3, 1 << 17, 3_300_002, 26, 3),
                                             (3, 1 << 17, 3_300_002, 48, 4), (5, 1 << 15, 3_100_003, 8, 2),
                                             (5, 1 << 15, 3_100_003, 30, 3)])
@pytest.mark.parametrize("W", [2, 4, 6, 8])
def test_cells_of_a_bundle(r, c, d, seed, sums, W):
    p = cs.cs_params_init(r, c, seed, d)
    residues = sum(p.visit[j].gmax for j in range(r))
    assert all(p.visit[j].K > 0 and p.visit[j].cost < p.visit[j].cost_walk for j in range(r))
    assert max(p.visit[j].ncell for j in range(r)) == sums
    assert r * d < 25 * residues and residues * 2 >= 2048 * 1024      # not a wavefront per vector; enough for runs of 16
    plain = cs.CsParams.from_buffer_copy(p)
    plain.flags |= B.CS_FLAG_NO_VISIT_LIST
    gen = torch.Generator(device=DEV).manual_seed(W)
    g = [torch.randint(-8, 9, (d,), device=DEV, generator=gen).float() for _ in range(W)]
    n = cs.cs_bundle_floats(p, W)
    want, got = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    cs.cs_sketch_accumulate_bundle(plain, want, g, i0=5, scale=0.5)
    cs.cs_sketch_accumulate_bundle(p, got, g, i0=5, scale=0.5)
    np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    S = torch.zeros(r, c, device=DEV)
    cs.cs_sketch_accumulate_sum(p, S, g, i0=5, scale=0.5)
    np.testing.assert_array_equal(S.cpu().numpy(), want.view(r, c, 8).sum(2).cpu().numpy())
