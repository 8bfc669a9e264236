"""The lists that one vector by itself is sketched along (up to 8 running sums a coordinate): they tile the vector and keep every
coordinate within their cells; vectors of small whole numbers, whose sums are exact, against the same call with the lists
switched off, bit for bit, into a table, into one worker's slot, of a length below the planned one, and along a list that
leads out of the cells it keeps."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

DEV = "cuda:0"
P61 = (1 << 61) - 1
SHAPES = [(5, 1 << 17, 3_000_001), (7, 1 << 16, 3_000_002), (5, 1 << 20, 25_000_003)]


@pytest.mark.parametrize("r,c,d", SHAPES)
def test_lists_stay_within_their_cells(r, c, d):
    p = cs.cs_params_init(r, c, 190304488, d)
    own = [j for j in range(r) if p.vector[j].list.K]
    assert own and any(p.vector[j].list.ncell > 4 for j in range(r)) == (c != 1 << 17)
    for j in range(r):
        assert p.vector[j].none == 0 and p.anyc[j].K == 0 and p.anyc[j].omega == 0
    for j in own:
        v = p.vector[j].list
        gaps = v.gaps()
        assert v.cover == d == sum(gaps) and max(gaps) == v.gmax and 2 <= v.ncell <= B.CS_VECTOR_CELLS
        s = 0
        for g in gaps:
            assert (p.a[j] * s % P61) % c + 1 < v.ncell, (j, s)
            s += g


@pytest.mark.parametrize("r,c,d", [(5, 1 << 20, 73_000_003), (5, 1 << 18, 25_000_001), (15, 8192, 1_300_001), (5, 250_007, 3_000_001)])
def test_kept_only_where_they_save_requests(r, c, d):
    p = cs.cs_params_init(r, c, 190304488, d)
    assert any(p.vector[j].list.K for j in range(r)) == (d == 73_000_003) if p.c_pow2 else any(p.anyc[j].K for j in range(r))


@pytest.mark.gpu
@pytest.mark.parametrize("forged", [False, True])
@pytest.mark.parametrize("r,c,planned", SHAPES + [(3, 1 << 20, 5_242_881), (7, 1 << 20, 8_388_609)])
def test_one_vector(r, c, planned, forged):
    p = cs.cs_params_init(r, c, 190304488, planned)
    plain = cs.CsParams.from_buffer_copy(p)
    plain.flags |= B.CS_FLAG_NO_VISIT_LIST
    if forged:                                         # more and fewer running sums than the offsets ask for
        for j in range(r):
            v = p.vector[j].list
            v.ncell = max(2, v.ncell - 2) if j % 2 else min(B.CS_VECTOR_CELLS, v.ncell + 1)
    for d in (planned, planned - 12_345):
        gen = torch.Generator(device=DEV).manual_seed(d)
        g = torch.randint(-8, 9, (d,), device=DEV, generator=gen).float()
        want, got = torch.zeros(r, c, device=DEV), torch.zeros(r, c, device=DEV)
        cs.cs_sketch_accumulate(plain, want, g, i0=7, scale=0.5)
        cs.cs_sketch_accumulate(p, got, g, i0=7, scale=0.5)
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
        T = torch.zeros(cs.cs_bundle_floats(p, 1), device=DEV)
        cs.cs_sketch_accumulate_bundle(p, T, [g], i0=7, scale=0.5)
        np.testing.assert_array_equal(T.view(r, c, 8)[:, :, 0].cpu().numpy(), want.cpu().numpy())
