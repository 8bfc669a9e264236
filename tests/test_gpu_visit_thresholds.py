"""Updates along visit lists tell a coordinate's cell and sign by comparing the top 32 bits of its hash with a
threshold of the visit.  Coordinates whose hash lies at such a threshold, or shares its top bits with it, have to
come out as the definition has them."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import paper_1903_04488_amd as cs
from oracle import cs_oracle as orc
from parity_util import assert_cells_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
P = (1 << 61) - 1
RESIDUE = 5


def _offsets(p, j):
    return np.concatenate([[0], np.cumsum((p.visit if p.c_pow2 else p.anyc)[j].gaps())[:-1]])


def _index_base(p, j, k, sign, below):
    """i0 such that the hash of coordinate RESIDUE, moved on by visit k, ends `below` short of p: 1 is the last
    value that does not wrap, 0 the first that does"""
    a, b = (p.as_[j], p.bs[j]) if sign else (p.a[j], p.b[j])
    A = a * int(_offsets(p, j)[k]) % P
    x = (P - A - below) % P
    return ((x - b) * pow(a, -1, P) - RESIDUE) % P


def _sketch(sk, g, i0):
    n = 1 << 18
    with ThreadPoolExecutor(max_workers=8) as pool:
        return sum(pool.map(lambda lo: sk.sketch(g[lo:lo + n], i0=i0 + lo), range(0, g.size, n)), sk.zeros())


# a power of two with two to four running sums, and one and two cells per wrap for other column counts
@pytest.mark.parametrize("r,c,d,seed", [(5, 1 << 15, 3_200_003, 31), (3, 5001, 1_000_003, 31), (3, 9001, 400_003, 47)])
@pytest.mark.parametrize("sign", [False, True])
@pytest.mark.parametrize("below", [1, 0, -(1 << 28), 1 << 28])
def test_update_at_the_thresholds(r, c, d, seed, sign, below):
    p = cs.cs_params_init(r, c, seed, d)
    sk = orc.SketchOracle(r, c, seed)
    j = r - 1
    lists = p.visit if p.c_pow2 else p.anyc
    assert all(lists[q].K > 0 for q in range(r))
    k = lists[j].K // 2
    i0 = _index_base(p, j, k, sign, below)
    if i0 > P - d:                                   # (not reachable with a global index)
        pytest.skip("index base beyond the range of the entry point")
    g = (np.random.default_rng(k).standard_normal(d) * 0.01).astype(np.float32)
    g[RESIDUE + int(_offsets(p, j)[k])] = 1.0        # a wrong cell or sign of this one is seen
    dev = torch.from_numpy(g).to(DEV)
    ref = _sketch(sk, g, i0)
    S = torch.zeros(r, c, dtype=torch.float32, device=DEV)
    cs.cs_sketch_accumulate(p, S, dev, i0=i0)
    assert_cells_close(S.cpu().numpy(), ref, terms_per_cell=d / c)
    for W in (2, 3, 8):                              # walkers of 2, 4 and 8 workers, the vector last among them
        gs = [torch.zeros_like(dev)] * (W - 1) + [dev]
        T = torch.zeros(cs.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV)
        cs.cs_sketch_accumulate_bundle(p, T, gs, i0=i0)
        assert_cells_close(T.view(r, c, cs.CS_BUNDLE_GROUP)[:, :, W - 1].cpu().numpy(), ref, terms_per_cell=d / c,
                           what=f"{W} workers")
        S.zero_()
        cs.cs_sketch_accumulate_sum(p, S, gs, i0=i0)
        assert_cells_close(S.cpu().numpy(), ref, terms_per_cell=d / c, what=f"sum of {W} workers")
