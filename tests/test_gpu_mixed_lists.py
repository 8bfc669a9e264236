"""Rows of both kinds of lists for any column count (2 and 4 running sums) in one launch of the update and of the query:
vectors of small whole numbers, whose sums are exact, against the same calls with the lists switched off, bit for bit."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _mixed(r, c, d, rows):
    """a sketch whose first `rows` rows hold lists of both kinds"""
    for seed in range(1, 200):
        p = cs.cs_params_init(r, c, seed, d)
        if all(p.anyc[j].K for j in range(r)) and {p.anyc[j].omega for j in range(rows)} == {1, 2}:
            plain = cs.CsParams.from_buffer_copy(p)
            plain.flags |= B.CS_FLAG_NO_VISIT_LIST
            return p, plain
    raise AssertionError("no such sketch")


# up to 5 rows groups of workers share a launch, 6 rows a launch takes, 7 go kind by kind (their query takes 6 together)
@pytest.mark.parametrize("r, c, d", [(3, 70_001, 1_600_003), (5, 70_001, 2_300_001), (7, 100_003, 1_700_001)])
def test_rows_of_both_kinds(r, c, d):
    p, plain = _mixed(r, c, d, r - 1)
    gen = torch.Generator(device=DEV).manual_seed(r)
    g = [torch.randint(-8, 9, (d,), device=DEV, generator=gen).float() for _ in range(17)]
    for W in (2, 4, 8, 9, 17):
        got, want = (torch.zeros(B.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV) for _ in range(2))
        cs.cs_sketch_accumulate_bundle(p, got, g[:W], i0=5)
        cs.cs_sketch_accumulate_bundle(plain, want, g[:W], i0=5)
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy(), err_msg=f"{W} workers")
    S = torch.randn(r, c, device=DEV, generator=gen)
    got, want = (torch.empty(d, dtype=torch.float32, device=DEV) for _ in range(2))
    ws = torch.empty(max(4, B.cs_estimate_scratch_bytes(p, d)), dtype=torch.uint8, device=DEV)
    counts = torch.empty(B.CS_TOPK_HIST_BINS, dtype=torch.int64, device=DEV)
    B.cs_sketch_estimate(p, S, got, 5, ws, counts)
    B.cs_sketch_estimate(plain, S, want, 5, None)
    np.testing.assert_array_equal(got.cpu().numpy().view(np.uint32), want.cpu().numpy().view(np.uint32))
    assert counts.sum().item() == d
