"""What HotPath does around the library's calls, without a GPU: the calls are recorded."""
import types

import pytest
import torch

from paper_1903_04488_amd import binding, pipeline


@pytest.fixture
def calls(monkeypatch):
    """names of the library calls that the pipeline makes, in order, with their arguments"""
    made = []
    fake = types.SimpleNamespace(**{n: getattr(binding, n) for n in dir(binding) if n.startswith("CS_")})
    fake.CsParams, fake.CsVisitPlan = binding.CsParams, binding.CsVisitPlan
    fake.DeviceVectors = lambda vectors, name=None: list(vectors)
    for name in dir(binding):
        if name.startswith("cs_"):
            setattr(fake, name, lambda *a, _name=name, **kw: made.append((_name, a, kw)))
    monkeypatch.setattr(pipeline, "B", fake)
    return made


def bare(cls=pipeline.HotPath, **attributes):
    """a path whose tensors are what the test gives it"""
    path = cls.__new__(cls)
    for name in ("params", "T", "S_t", "S_u", "S_v", "est", "est_ws", "cand", "est_at_cand", "x_cand", "idx", "x",
                 "delta", "uhat", "topk_ws", "_counts"):
        setattr(path, name, None)
    path.d, path.W, path.r, path.c, path.k, path.kq, path.P = 100_000, 4, 5, 64, 2, 2, 1
    path.rho, path.fold_workers, path.device = 0.9, False, torch.device("cpu")
    for name, value in attributes.items():
        setattr(path, name, value)
    return path


def names(made):
    return [name for name, _, _ in made]


def test_a_step_runs_the_stages_that_a_subclass_overrides(calls):
    class Reduced(pipeline.HotPath):
        def merge(self):
            calls.append(("all-reduce", (), {}))

    class Plain(pipeline.HotPath):
        def momentum(self):
            calls.append(("no momentum", (), {}))

    bare().step([None])
    assert "cs_bundle_merge_momentum" in names(calls)
    calls.clear()
    bare(Reduced).step([None])
    assert names(calls).count("all-reduce") == 1 and "cs_sketch_momentum" in names(calls)
    assert "cs_bundle_merge_momentum" not in names(calls)
    calls.clear()
    bare(Plain).step([None])
    assert "cs_bundle_merge" in names(calls) and names(calls).count("no momentum") == 1
    assert "cs_bundle_merge_momentum" not in names(calls) and "cs_sketch_momentum" not in names(calls)
    calls.clear()
    path = bare()
    path.merge = lambda: calls.append(("wrapped", (), {}))           # on the object itself
    path.step([None])
    assert "wrapped" in names(calls) and "cs_bundle_merge_momentum" not in names(calls)
    calls.clear()
    bare(pipeline.ReproduciblePath, acc=torch.zeros(1), frac_bits=40, dropped=None, S_fb=None).step([None])
    assert "cs_fixed_to_float" in names(calls) and "cs_bundle_merge_momentum" not in names(calls)


def test_the_vectors_of_a_step_reach_overridden_stages_as_a_sequence_of_tensors(calls, monkeypatch):
    monkeypatch.setattr(pipeline.B, "DeviceVectors", binding.DeviceVectors)
    monkeypatch.setattr(binding, "_ptr_array", lambda tensors, dtype, name, numel=None: None)   # (host tensors here)
    seen = []

    class Stacked(pipeline.HotPath):
        def accumulate(self, g_w):
            seen.append(torch.stack(g_w).sum(0))
            seen.append([g + 1 for g in g_w[1:]])

    bare(Stacked).step([torch.ones(3), torch.full((3,), 2.0)])
    assert seen[0].tolist() == [3.0, 3.0, 3.0] and len(seen[1]) == 1 and seen[1][0].tolist() == [3.0, 3.0, 3.0]


@pytest.mark.parametrize("scratch", [0, 4 * 100_000, 20 * 100_000])
@pytest.mark.parametrize("W,given,length", [(4, 4, 100_000), (1, 3, 100_000), (1, 1, 100_000), (4, 3, 70_000),
                                            (4, 4, 130_000)])
def test_folded_workers_are_all_summed_whenever_folding_was_chosen(calls, W, given, length, scratch):
    """fold_workers set on a finished object, more vectors than W said, vectors of another length than d"""
    path = bare(W=W, est_ws=torch.empty(scratch, dtype=torch.uint8) if scratch else None, g_mean=None)
    path.fold_workers = True
    vectors = [torch.full((length,), float(w)) for w in range(given)]
    path.accumulate(vectors)
    made = [(name, a, kw) for name, a, kw in calls if name != "cs_sketch_zero"]
    if given == 1:
        assert names(made) == ["cs_sketch_accumulate"] and made[0][1][2] is vectors[0]
        assert made[0][2].get("scale", 1.0) == 1.0 / W
        return
    assert names(made) == ["cs_vectors_sum", "cs_sketch_accumulate"]
    (x_w, out), kw = made[0][1], made[0][2]
    assert len(x_w) == given and kw["alpha"] == 1.0 / W
    assert out.numel() == length and out.dtype == torch.float32 and made[1][1][2] is out
    if scratch >= 4 * length and length <= path.d:                   # no memory of its own where the query has scratch
        assert out.data_ptr() == path.est_ws.data_ptr()


@pytest.mark.parametrize("scratch,need,built", [(5000, 4000, True), (0, 4000, True), (5000, 5001, False),
                                                (5000, 4600, False), (5000, 4500, True)])
@pytest.mark.parametrize("fold", [False, True])
def test_running_sums_have_memory_of_their_own_up_to_a_limit(monkeypatch, fold, scratch, need, built):
    """whatever the query's scratch takes, and not in it"""
    monkeypatch.setattr(pipeline.B, "cs_update_index_bytes", lambda p, W, d: 64)
    monkeypatch.setattr(pipeline.B, "cs_update_workspace_bytes", lambda p, W, d: need)
    monkeypatch.setattr(pipeline.B, "cs_update_index_build", lambda p, d, index: None)
    monkeypatch.setattr(pipeline.HotPath, "SUMS_OWN_BYTES", 4500)
    path = bare(fold_workers=fold, d=100, params=binding.CsParams(),
                est_ws=torch.empty(scratch, dtype=torch.uint8) if scratch else None)
    path._build_index()
    assert (path._index is not None) == built
    if built and scratch:
        ws, own = path._sums_ws, path.est_ws
        assert ws.numel() == need
        assert ws.data_ptr() + need <= own.data_ptr() or own.data_ptr() + scratch <= ws.data_ptr()


@pytest.mark.parametrize("limit,built", [(0, False), (63, False), (64, True), (None, True)])
@pytest.mark.parametrize("fold", [False, True])
def test_cell_lists_are_bounded_by_the_limit_of_a_path_s_own_memory(monkeypatch, fold, limit, built):
    monkeypatch.setattr(pipeline.B, "cs_cell_lists_bytes", lambda p, W, d: 64)
    monkeypatch.setattr(pipeline.B, "cs_cell_lists_build", lambda p, d, lists: None)
    if limit is not None:
        monkeypatch.setattr(pipeline.HotPath, "SUMS_OWN_BYTES", limit)
    path = bare(fold_workers=fold, d=100, params=binding.CsParams())
    assert path._build_cell_lists() == built == path._cell_lists and (path._index is not None) == built


@pytest.mark.parametrize("index", [False, True])
def test_tables_of_workers_may_be_made_beside_the_query_of_the_step_before(calls, monkeypatch, index):
    """accumulate alone, workers not folded: no memory that it is given is the query's"""
    def memory(n):
        return torch.empty(n, dtype=torch.uint8)
    path = with_index(monkeypatch, S_t=memory(9), S_u=memory(9), S_v=memory(9), T=memory(9), est=memory(9), est_ws=memory(9),
                      _counts=memory(9), d=100_000, params=binding.cs_params_init(5, 64, 3, 100_000))
    if not index:
        path._index = None
    path.accumulate([torch.zeros(path.d)] * path.W)
    assert ("cs_bundle_sketch" in names(calls)) == index
    given = [t for _, a, kw in calls for t in (*a, *kw.values())]
    given = [t for g in given for t in (g if isinstance(g, (list, tuple)) else [g]) if isinstance(t, torch.Tensor)]
    calls.clear()
    path.estimate()
    query = [t for _, a, kw in calls for t in (*a, *kw.values()) if isinstance(t, torch.Tensor)]
    assert len(query) == 4                               # the table asked, est, scratch, counts
    assert path.T.data_ptr() in {t.data_ptr() for t in given}
    assert not {t.data_ptr() for t in given} & {t.data_ptr() for t in query}


def with_index(monkeypatch, cls=pipeline.HotPath, **attributes):
    """a path that has an index for what it holds now; building it is not among the recorded calls"""
    attributes = {"params": binding.cs_params_init(5, 64, 3, 5000), "d": 5000, "W": 2, **attributes}
    path = bare(cls, **attributes)
    with monkeypatch.context() as m:
        m.setattr(pipeline.B, "cs_update_index_bytes", lambda p, W, d: 64)
        m.setattr(pipeline.B, "cs_update_workspace_bytes", lambda p, W, d: 64)
        m.setattr(pipeline.B, "cs_update_index_build", lambda p, d, index: None)
        path._build_index()
    return path


def no_lists(path):
    path.params.flags |= binding.CS_FLAG_NO_VISIT_LIST


def hash_constant(path):
    path.params.b[4] += 1


@pytest.mark.parametrize("change", [
    lambda path: setattr(path, "params", binding.cs_params_init(5, 64, 4, 5000)), no_lists, hash_constant,
    lambda path: setattr(path, "W", 3), lambda path: setattr(path, "d", 4999),
    lambda path: setattr(path, "fold_workers", not path.fold_workers)])
@pytest.mark.parametrize("fold", [False, True])
def test_an_index_serves_what_it_was_made_for_alone(calls, monkeypatch, fold, change):
    """another sketch's cells have other sums, another length or number of vectors another workspace"""
    path = with_index(monkeypatch, fold_workers=fold, g_mean=None)
    path.step([torch.zeros(path.d)] * path.W)
    path.accumulate([torch.zeros(path.d)] * path.W)
    assert names(calls).count("cs_bundle_sketch") == 2
    calls.clear()
    path.params = binding.CsParams.from_buffer_copy(path.params)     # (equal ones are the same sketch)
    path.accumulate([torch.zeros(path.d)] * path.W)
    assert names(calls).count("cs_bundle_sketch") == 1
    calls.clear()
    change(path)
    vectors = [torch.zeros(path.d)] * path.W
    path.step(vectors)
    path.accumulate(vectors)
    if path.fold_workers and path.W != 2 and path.d == 5000:          # (folded: one vector, their sum, either way)
        assert names(calls).count("cs_bundle_sketch") == 2
        return
    assert "cs_bundle_sketch" not in names(calls)
    assert names(calls).count("cs_sketch_accumulate" if path.fold_workers else "cs_sketch_accumulate_bundle") == 2


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("rho", [0.9, 0.0, None])
def test_state_is_advanced_while_the_path_has_a_momentum_factor(calls, monkeypatch, fold, rho):
    """rho set on a finished path, with an index as without one: None leaves S_u and S_v alone"""
    path = with_index(monkeypatch, fold_workers=fold, g_mean=None, S_t="S_t", S_u="S_u", S_v="S_v")
    path.rho = rho
    path.sketch_and_aggregate([torch.zeros(path.d)] * path.W)
    assert "cs_bundle_sketch" in names(calls) and "cs_sketch_momentum" not in names(calls)
    tables = next(kw for name, _, kw in calls if name == "cs_bundle_sketch")
    assert tables["S_t"] == "S_t"
    if rho is None:
        assert tables.get("S_u") is None and tables.get("S_v") is None
    else:
        assert (tables["S_u"], tables["S_v"], tables["rho"]) == ("S_u", "S_v", rho)


# shapes on both sides of every line of the rule, each where it was measured to be the faster one (W = 0: one vector)
@pytest.mark.parametrize("W,d,r,c,two_passes", [
    (1, 2_000_000, 5, 65_536, True), (4, 1 << 20, 5, 1 << 15, True), (4, 16_000_000, 5, 1 << 15, False),
    (4, 9_054_897, 5, 1 << 14, False), (4, 20_279_047, 3, 1 << 19, True), (4, 9_378_155, 15, 65_536, False),
    (4, 7_062_633, 5, 65_536, True), (3, 18_219_159, 3, 1 << 15, True), (3, 22_656_597, 3, 65_536, False),
    (16, 300_000, 5, 4096, True), (16, 1 << 20, 5, 1 << 15, True), (11, 2_244_359, 5, 4096, False),
    (12, 1_353_347, 5, 8192, False), (7, 358_975, 15, 8192, True), (5, 75_740, 7, 1024, False), (15, 46_637, 7, 1024, False),
    (14, 123_444, 5, 1024, True), (6, 18_193, 15, 1024, True), (8, 212_744, 5, 512, True), (14, 39_685, 5, 64, True),
    (2, 11_187, 5, 64, False), (11, 10_840, 5, 64, False), (13, 24_449, 5, 64, True), (15, 5844, 7, 64, True),
    (0, 2_600_000, 5, 65_536, True), (0, 460_000, 5, 4096, False), (0, 795_397, 15, 8192, False),
    (0, 1_085_510, 15, 8192, True)])
def test_the_way_of_an_update_is_the_faster_one(W, d, r, c, two_passes):
    p = binding.cs_params_init(r, c, 190304488, d)
    assert binding.cs_update_workspace_bytes(p, max(W, 1), d) > 0
    assert (binding.cs_update_index_bytes(p, W, d) > 0) == two_passes


@pytest.mark.parametrize("d", [784, 32_768, 32_769])
def test_counts_by_magnitude_are_there_for_vectors_of_any_length(calls, d):
    """up to CS_TOPK_SMALL_D neither the estimate nor the selection is given the counts; whoever reads
    them gets those of the estimates all the same"""
    est = torch.randn(d, generator=torch.Generator().manual_seed(d))
    counts = torch.full((binding.CS_TOPK_HIST_BINS,), 7, dtype=torch.int64)
    path = bare(hist=counts)
    path.d, path.est = d, est
    path.estimate()
    path.topk()
    given = calls[0][1][-1]
    assert (given is None) == (d <= binding.CS_TOPK_SMALL_D) and calls[1][1][-1] is given
    if given is not None:
        assert given is counts and path.hist is counts
        return
    bins = (est.numpy().view("uint32") & 0x7FFFFFFF) >> 20
    assert path.hist is counts
    assert counts.tolist() == torch.bincount(torch.from_numpy(bins.astype("int64")), minlength=2048).tolist()


def test_a_step_shares_launches_only_between_stages_that_are_its_own(calls):
    shared = {"cs_sketch_estimate_topk", "cs_gather_feedback"}
    short = dict(d=100, est=torch.empty(100), params=types.SimpleNamespace(r=5))
    bare(**short).step([None])
    assert shared <= set(names(calls)) and "cs_gather_exact" not in names(calls)
    for stage, call in (("estimate", "cs_sketch_estimate_topk"), ("topk", "cs_sketch_estimate_topk"),
                        ("gather", "cs_gather_feedback"), ("feedback", "cs_gather_feedback")):
        calls.clear()
        path = bare(**short)
        setattr(path, stage, lambda *a: calls.append(("own", (), {})))
        path.step([None])
        assert "own" in names(calls) and call not in names(calls) and shared - {call} <= set(names(calls))
    for other in (dict(d=2000, est=torch.empty(2000)), dict(est=torch.empty(2000)), dict(params=types.SimpleNamespace(r=99))):
        calls.clear()
        bare(**{**short, **other}).step([None])
        assert "cs_sketch_estimate_topk" not in names(calls) and "cs_heavy_hitters_topk_kept" in names(calls)
    calls.clear()
    bare(**short, idx=torch.empty(1)).step([None])             # (candidates and selection apart)
    assert "cs_gather_feedback" not in names(calls) and "cs_sketch_feedback_pair" in names(calls)
    calls.clear()
    bare(**{**short, "rho": None}).step([None])
    assert "cs_gather_feedback" not in names(calls) and "cs_gather_exact" in names(calls)
