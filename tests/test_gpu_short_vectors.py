"""The forms that short vectors and single vectors take (visit chains in pieces, one-vector update, the
sum of folded workers) at the edges of their tiles."""
import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc
from parity_util import assert_cells_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("W", [1, 2, 4, 8, 9])
@pytest.mark.parametrize("r,c,d", [(7, 256, 30_403), (5, 64, 4097), (5, 1 << 12, 255_999), (3, 771, 66_281)])
def test_updates_of_short_vectors(W, r, c, d):
    p = cs.cs_params_init(r, c, 190304488, d)
    sk = orc.SketchOracle(r, c, 190304488)
    rng = np.random.default_rng(d + W)
    gs = [(rng.standard_normal(d) * 0.01).astype(np.float32) for _ in range(W)]
    dev = [torch.from_numpy(g).to(DEV) for g in gs]
    T = torch.zeros(cs.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV)
    cs.cs_sketch_accumulate_bundle(p, T, dev)
    G = cs.CS_BUNDLE_GROUP
    got = T.cpu().numpy().reshape(-1, r, c, G)
    for w in range(W):
        assert_cells_close(got[w // G, :, :, w % G], sk.sketch(gs[w]), terms_per_cell=d / c, what=f"worker {w}")
    S = torch.zeros(r, c, dtype=torch.float32, device=DEV)
    cs.cs_sketch_accumulate(p, S, dev[0], i0=5, scale=0.5)
    assert_cells_close(S.cpu().numpy(), sk.sketch(gs[0], i0=5, scale=0.5), terms_per_cell=d / c)


@pytest.mark.parametrize("W", [1, 3, 4, 257])
@pytest.mark.parametrize("d", [1, 1023, 4100])
def test_vectors_sum(W, d):
    x = torch.randn(W, d, generator=torch.Generator().manual_seed(W)).to(DEV)
    out = torch.empty(d, dtype=torch.float32, device=DEV)
    cs.cs_vectors_sum([x[w] for w in range(W)], out, alpha=1.0 / W)
    torch.testing.assert_close(out.cpu(), x.cpu().double().mean(0).float(), rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("offset", [0, 1])
def test_vectors_sum_of_large_values_above_one_launch(offset):
    """The mean of 300 vectors of 2e36 is finite though their sum is not: the part that the first launch
    (256 vectors) leaves in `out` is scaled already."""
    W, d = 300, 1029
    g = torch.Generator().manual_seed(7)
    x = (torch.rand(W, d + offset, generator=g) + 0.5) * 2e36
    dev = [x[w].to(DEV)[offset:] for w in range(W)]
    out = torch.empty(d, dtype=torch.float32, device=DEV)
    cs.cs_vectors_sum(dev, out, alpha=1.0 / W)
    # two partial means, each rounded once, and their sum
    torch.testing.assert_close(out.cpu(), x[:, offset:].double().mean(0).float(), rtol=3 * 2.0 ** -24, atol=0.0)
