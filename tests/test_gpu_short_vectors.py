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


@pytest.mark.parametrize("W", [1, 3, 5])
@pytest.mark.parametrize("d", [1, 3, 4, 1029])
@pytest.mark.parametrize("odd", ["inputs", "one input", "output"])
def test_vectors_sum_at_any_dword_address(W, d, odd):
    """views that begin 4, 8 or 12 bytes past a 16-byte boundary; nothing around `out` is written"""
    x = torch.randn(W, d, generator=torch.Generator().manual_seed(W * d))
    views = []
    for w in range(W):
        shift = (1 + w % 3) if odd == "inputs" or (odd == "one input" and w == W - 1) else 0
        buf = torch.zeros(d + 8, dtype=torch.float32, device=DEV)
        views.append(buf[shift:shift + d])
        views[-1].copy_(x[w])
    shift = 2 if odd == "output" else 0
    buf = torch.full((d + 8,), 7.0, dtype=torch.float32, device=DEV)
    cs.cs_vectors_sum(views, buf[shift:shift + d], alpha=0.5)
    # exact sums in binary64, scaled by a power of two, rounded once
    np.testing.assert_array_equal(buf[shift:shift + d].cpu().numpy(), (0.5 * x.double().sum(0)).float().numpy())
    assert (buf[:shift] == 7.0).all() and (buf[shift + d:] == 7.0).all()


@pytest.mark.parametrize("W", [1, 8, 9, 40])
@pytest.mark.parametrize("r,c", [(3, 1), (5, 1 << 10), (7, 771)])
def test_bundle_merge_with_momentum(W, r, c):
    p = cs.cs_params_init(r, c, 3)
    rng = np.random.default_rng(W + c)
    G = cs.CS_BUNDLE_GROUP
    T = rng.standard_normal((-(-W // G), r, c, G)).astype(np.float32)
    if W % G:
        T[-1, :, :, W % G:] = 0.0                                    # padding slots
    su, sv = (rng.standard_normal((r, c)).astype(np.float32) for _ in range(2))
    S_t = torch.full((r, c), float("nan"), dtype=torch.float32, device=DEV)
    S_u, S_v = torch.from_numpy(su).to(DEV), torch.from_numpy(sv).to(DEV)
    alpha = float(np.float32(1.0 / W))
    cs.cs_bundle_merge_momentum(p, S_t, S_u, S_v, torch.from_numpy(T.reshape(-1)).to(DEV), W, alpha, 0.9)
    merged = orc.merge([T[w // G, :, :, w % G] for w in range(W)], alpha=alpha)
    st = orc.SketchSpaceState(orc.SketchOracle(r, c, 3), 0.9)
    st.S_u, st.S_v = su.astype(np.float64), sv.astype(np.float64)
    st.momentum(merged)
    # the merge is rounded once, the momentum twice more and the accumulation once more, each to 2^-24 of
    # an operand: four roundings of values below |S_t| + |S_u| + |S_v|
    bound = 4 * 2.0 ** -24 * (np.abs(merged) + np.abs(su) + np.abs(sv))
    for got, want, name in ((S_t, merged, "S_t"), (S_u, st.S_u, "S_u"), (S_v, st.S_v, "S_v")):
        assert (np.abs(got.cpu().numpy() - want) <= bound).all(), name


def _listed(p, d, forged):
    """the lists of p, or lists of evenly spaced visits that keep no coordinate within its cells; either
    way short enough in residues that the update of one vector follows them"""
    import ctypes
    P = (1 << 61) - 1
    plans = p.visit if p.c_pow2 else p.anyc
    for j in range(p.r if forged else 0):
        v, K = plans[j], 40
        ctypes.memset(ctypes.byref(v), 0, ctypes.sizeof(v))
        gap = d // K - j
        last = d - (K - 1) * gap
        v.K, v.cover, v.gmax, v.cost = K, d, max(gap, last), 1
        if p.c_pow2:
            v.ncell, v.cost_walk = 2 + j % 3, 2
            v.gap[0], v.gap[3] = gap, last
            v.A[0], v.As[0] = (p.a[j] * gap) % P, (p.as_[j] * gap) % P
            v.code[(K - 1) // 16] |= 3 << (2 * ((K - 1) % 16))       # the last visit: code 3
        else:
            v.omega, v.cost_direct = 1 + j % 2, 2
            for k in range(K):
                v.gap[k] = gap if k + 1 < K else last
    assert all(v.K > 0 and v.cover >= d and v.cost < (v.cost_walk if p.c_pow2 else v.cost_direct) for v in plans[:p.r])
    assert 1.2 * sum(plans[j].gmax for j in range(p.r)) <= p.r * d / 8
    return p


@pytest.mark.parametrize("r,c,d", [(5, 1 << 12, 200_003), (3, 5001, 1_000_003), (5, 1 << 15, 3_000_003)])
@pytest.mark.parametrize("forged", [False, True])
def test_update_of_one_vector_with_nan_infinities_and_forged_lists(r, c, d, forged):
    """Into a table of its own, into a slot of a bundle (the ninth worker), and summed: a NaN or an
    infinity reaches the r cells of its coordinate and no others, and a wrong list costs time only."""
    p = _listed(cs.cs_params_init(r, c, 11, d), d, forged)
    sk = orc.SketchOracle(r, c, 11)
    rng = np.random.default_rng(c)
    g = (rng.standard_normal(d) * 0.01).astype(np.float32)
    g[[7, 30_001]] = [np.nan, np.inf]
    g[[50_000, 50_001, d - 1]] = [-np.inf, np.inf, np.nan]
    plain = (rng.standard_normal(d) * 0.01).astype(np.float32)
    G = cs.CS_BUNDLE_GROUP
    for vec in (plain, g):
        with np.errstate(invalid="ignore"):
            ref = sk.sketch(vec, i0=3, scale=0.5)
        dev = torch.from_numpy(vec).to(DEV)
        S = torch.zeros(r, c, dtype=torch.float32, device=DEV)
        cs.cs_sketch_accumulate(p, S, dev, i0=3, scale=0.5)
        S_sum = torch.zeros(r, c, dtype=torch.float32, device=DEV)
        cs.cs_sketch_accumulate_sum(p, S_sum, [dev], i0=3, scale=0.5)
        T = torch.zeros(cs.cs_bundle_floats(p, 9), dtype=torch.float32, device=DEV)
        cs.cs_sketch_accumulate_bundle(p, T, [torch.ones_like(dev)] * 8 + [dev], i0=3, scale=0.5)
        for table in (S, S_sum, T.view(-1, r, c, G)[1, :, :, 0]):
            got = table.cpu().numpy()
            np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
            np.testing.assert_array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(ref), ref, 0))
            fin = np.isfinite(ref)
            assert fin.sum() >= ref.size - 5 * r
            assert_cells_close(np.where(fin, got, 0), np.where(fin, ref, 0), terms_per_cell=d / c)


@pytest.mark.parametrize("r,c", [(3, 1 << 14), (5, 1 << 16)])
@pytest.mark.parametrize("below", [0, 1])
def test_update_of_one_vector_where_its_two_forms_meet(r, c, below):
    """r d = 15 million: from there on along visit lists, below as a lattice"""
    d = 15_000_000 // r - below
    p = cs.cs_params_init(r, c, 21, d)
    g = torch.randn(d, generator=torch.Generator().manual_seed(d)) * 0.01
    S = torch.full((r, c), 0.25, dtype=torch.float32, device=DEV)
    cs.cs_sketch_accumulate(p, S, g.to(DEV), i0=11, scale=-0.5)
    ref = sketch_in_slices_from(orc.SketchOracle(r, c, 21), g.numpy(), 11)
    assert_cells_close(S.cpu().numpy(), 0.25 - 0.5 * ref, terms_per_cell=d / c)


def sketch_in_slices_from(sk, g, i0):
    from concurrent.futures import ThreadPoolExecutor
    n = 1 << 19
    with ThreadPoolExecutor(max_workers=8) as pool:
        return sum(pool.map(lambda lo: sk.sketch(g[lo:lo + n], i0=i0 + lo), range(0, g.size, n)), sk.zeros())


# Kernels that hash every coordinate take one or 8 of them a thread: one thread and a remainder, both sides of where 8
# begin for the query (2^18 coordinates, 196 608 with few cells) and for the tables (2^15, shared by the groups of workers; with several groups from 75
# coordinates per column on where there are fewer than 80, from 50 on with more than 8 rows).
@pytest.mark.parametrize("r,c,d,W", [(7, 40, 1, 1), (5, 97, 31, 3), (5, 257, 33, 9), (3, 4099, 32_767, 1), (3, 4099, 32_768, 1),
                                     (3, 4099, 16_383, 9), (3, 4099, 16_385, 9), (9, 4099, 262_143, 1), (3, 4099, 262_145, 2),
                                     (3, 33, 2474, 9), (3, 33, 2475, 9), (5, 79, 6001, 41), (15, 99, 4949, 10), (15, 99, 4950, 10),
                                     (5, 257, 196_607, 1), (5, 257, 196_609, 1)])
def test_coordinates_per_thread(r, c, d, W):
    p = cs.cs_params_init(r, c, 5, d)
    sk = orc.SketchOracle(r, c, 5)
    rng = np.random.default_rng(d)
    gs = [(rng.standard_normal(d) * 0.01).astype(np.float32) for _ in range(W)]
    T = torch.zeros(cs.cs_bundle_floats(p, W), dtype=torch.float32, device=DEV)
    cs.cs_sketch_accumulate_bundle(p, T, [torch.from_numpy(g).to(DEV) for g in gs])
    got = T.cpu().numpy().reshape(-1, r, c, cs.CS_BUNDLE_GROUP)
    for w in range(W):
        assert_cells_close(got[w // 8, :, :, w % 8], sk.sketch(gs[w]), terms_per_cell=max(1.0, d / c), what=f"worker {w}")
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(d)).to(DEV)
    est, want = torch.full((d + 1,), 77.0, device=DEV), torch.empty(d, device=DEV)
    cs.cs_sketch_estimate(p, S, est[:d], 3)
    cs.cs_sketch_estimate_sparse(p, S, torch.arange(3, d + 3, device=DEV), want)
    assert torch.equal(est[:d], want) and est[d] == 77.0


# sums of squares by rows, whole rounds of loads, remainders and rows at any address; their median, with NaN where the
# insertion sort that defines it leaves them
@pytest.mark.parametrize("r", [1, 3, 5, 15])
@pytest.mark.parametrize("c", [5, 1023, 8192, 8197, 32_768 + 4, 40_001])
@pytest.mark.parametrize("special", [None, "inf", "nan"])
def test_row_norms_and_their_median(r, c, special):
    p = cs.cs_params_init(r, c, 5, 100)
    S = torch.randn(r, c, generator=torch.Generator().manual_seed(c))
    if r > 1:
        S[-1] = S[0]                                  # two equal rows
    if special:
        S[r // 2, c - 1] = float(special)
    out = torch.empty(1 + r, dtype=torch.float64, device=DEV)
    cs.cs_sketch_l2sq(p, S.to(DEV), out)
    got = out.cpu().numpy()
    want = (S.double() ** 2).sum(1).numpy()
    # binary64 sums in another order: c 2^-53 at most
    np.testing.assert_allclose(got[1:], want, rtol=c * 2.0 ** -53, equal_nan=True)
    v = []
    for x in got[1:]:
        q = len(v)
        while q > 0 and v[q - 1] > x:
            q -= 1
        v.insert(q, x)
    np.testing.assert_equal(got[0], v[r // 2])
