"""More sketches in turn than the launches remember amounts of LDS for, and one whose rows take two launches of different amounts:
vectors of small whole numbers, whose sums are exact, against the update with the lists switched off, bit for bit, twice round."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_sketches_in_turn():
    W, rounds = 3, []
    gen = torch.Generator(device=DEV).manual_seed(1)
    for q in range(12):
        r, c, d = (15 if q == 5 else 5), 1 << 12, 100_003 + 17_001 * q
        p = cs.cs_params_init(r, c, 190304488 + q, d)
        assert all(p.visit[j].K > 0 for j in range(r))
        plain = cs.CsParams.from_buffer_copy(p)
        plain.flags |= B.CS_FLAG_NO_VISIT_LIST
        g = [torch.randint(-8, 9, (d,), device=DEV, generator=gen).float() for _ in range(W)]
        want = torch.zeros(cs.cs_bundle_floats(p, W), device=DEV)
        cs.cs_sketch_accumulate_bundle(plain, want, g)
        rounds.append((p, g, want))
    for _ in range(2):
        for p, g, want in rounds:
            got = torch.zeros_like(want)
            cs.cs_sketch_accumulate_bundle(p, got, g)
            np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
