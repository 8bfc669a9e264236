"""Cases of work that a program built on this framework has it do, for timing.

A case is one pass of one role in Sketched-SGD training, through the public entry points:

    step      HotPath.step: W workers' gradients sketched, merged, queried, selected, second round
              (with momentum and error feedback in sketch space when `rho` is not 0)
    graph     the same step replayed from a HIP graph (GraphedStep)
    fold      HotPath(fold_workers=True).step: the workers of the device summed as they are sketched
    dense     DenseStatePath.step: Alg. 3 as printed, dense momentum and error vectors per worker
    heavymix  Alg. 1's selection on the merged sketch (norm estimate, threshold, random fill)
    encode    one worker of a distributed job: sketch of its own gradient, in 16 bits for the wire
    decode    the aggregating side of a distributed job: W received tables merged, momentum and
              error accumulation, query of every coordinate, selection, feedback

Gradients are N(0, 0.01) noise, drawn per worker, plus as many heavy coordinates +-U(0.5, 1), shared by
the workers, as coordinates are selected.
"""
from __future__ import annotations

import math

import torch

from paper_1903_04488_amd import binding as B
from paper_1903_04488_amd.pipeline import DenseStatePath, GraphedStep, HotPath

DEV = "cuda:0"
HASH_SEED = 190304488
RHO = 0.9


def _case(kind, d, W, r, c, k, rho=0.0, P=1, name=None):
    case = {"kind": kind, "d": d, "W": W, "r": r, "c": c, "k": k, "rho": rho, "P": P}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest model: a sketch of 7 x 40 over 784 parameters; nothing but launches and host work
        _case("step", 784, 4, 7, 40, 2, RHO, name="step-784"),
        # a small model, the step called stage by stage, and the same step as a training loop that
        # is bound by its launches would run it
        _case("step", 1 << 20, 4, 5, 1 << 15, 1000, name="step-1M"),
        _case("graph", 1 << 20, 4, 5, 1 << 15, 1000, name="graph-1M"),
        # an LSTM-sized model
        _case("step", 6_500_000, 8, 5, 1 << 17, 5000, name="step-6.5M"),
        # a column count that is no power of two, as the paper's sketches have, an odd length, and the
        # selection of Alg. 1
        _case("heavymix", 6_500_003, 8, 5, 180_000, 5000, name="heavymix-6.5M"),
        # a residual-network-sized model with dense state on every worker
        _case("dense", 11_000_000, 8, 5, 1 << 18, 10_000, RHO, name="dense-11M"),
        # several workers on one device that need no tables of their own
        _case("fold", 25_000_000, 32, 5, 1 << 19, 10_000, RHO, name="fold-25M"),
        # the two sides of a distributed job: one worker's gradient to a 16-bit table, and the
        # tables of 16 workers to the selected coordinates (odd lengths)
        _case("encode", 73_000_003, 1, 5, 1 << 20, 0, name="encode-73M"),
        _case("decode", 11_000_003, 16, 5, 1 << 18, 5000, RHO, name="decode-11M"),
        # the paper's transformer sketch: 15 x 180 000 over 90 M parameters, 16 candidates per coordinate
        _case("step", 90_000_000, 4, 15, 180_000, 20_000, RHO, P=16, name="step-90M-15x180k"),
        # the headline configuration: a transformer-sized model, 32 workers
        _case("step", 100_000_000, 32, 5, 1 << 20, 20_000, RHO, name="step-100M"),
        # many workers
        _case("step", 25_000_000, 256, 7, 1 << 19, 10_000, RHO, name="step-25M-256w"),
    ]


def draw(rng):
    """One more case: every kind, vectors of 800 to 10^8 coordinates, 1 to 256 workers, sketches of
    3 to 15 rows with 1/20 to 1/500 as many columns as coordinates, a power of two or not."""
    kind = rng.choice(["step", "step", "step", "graph", "fold", "dense", "heavymix", "encode", "decode"])
    d = int(math.exp(rng.uniform(math.log(800), math.log(1e8))))
    # the whole job reads at most 3.2 G coordinates
    most = 16 if kind == "dense" else min(256.0, 3.2e9 / d)
    W = 1 if kind == "encode" else max(1, int(math.exp(rng.uniform(0.0, math.log(max(1.0, min(most, 3.2e9 / d)))))))
    columns = d / math.exp(rng.uniform(math.log(20), math.log(500)))
    columns = min(max(columns, 32.0), float(1 << 20))
    if rng.random() < 0.7:
        c = 1 << max(5, round(math.log2(columns)))
    else:
        c = max(33, int(columns)) | 1
    # (15 rows: the update reads a vector 15 times, so for jobs of up to 1.2 G coordinates only)
    r = rng.choice([3, 5, 5, 7, 15] if kind != "encode" and W * d < 1.2e9 else [3, 5, 5, 7])
    # (error feedback through a sketch with few columns per selected coordinate, or with 3 rows,
    # diverges when it is fed one gradient for long)
    k = max(1, int(c / math.exp(rng.uniform(math.log(40), math.log(400)))))
    if kind == "decode":
        r = max(r, 5)
    P = rng.choice([1, 1, 4, 16]) if kind in ("step", "fold") else 1
    if kind in ("dense", "decode"):
        rho = RHO
    else:
        rho = 0.0 if kind in ("heavymix", "encode") or r == 3 else rng.choice([0.0, RHO])
    return _case(kind, d, W, r, c, 0 if kind == "encode" else k, rho, P)


# ------------------------------------------------------------------------------------------
def _gradients(case, seed):
    d, W = case["d"], case["W"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    n = max(1, case["k"])
    # one heavy coordinate somewhere in each of n equal parts of the vector
    idx = ((torch.arange(n, device=DEV, dtype=torch.float64)
            + torch.rand(n, device=DEV, dtype=torch.float64, generator=gen)) * (d / n)).long().clamp_(max=d - 1)
    val = torch.empty(n, device=DEV).uniform_(0.5, 1.0, generator=gen)
    val *= torch.randint(0, 2, (n,), device=DEV, generator=gen) * 2 - 1
    g_w = []
    for _ in range(W):
        g = torch.empty(d, device=DEV).normal_(0.0, 0.01, generator=gen)
        g[idx] += val
        g_w.append(g)
    return g_w


class _State:
    pass


def prepare(case, seed):
    kind, d, W, r, c, k = (case[x] for x in ("kind", "d", "W", "r", "c", "k"))
    rho = case["rho"] or None
    s = _State()
    s.kind, s.k = kind, k
    f32 = dict(dtype=torch.float32, device=DEV)
    if kind == "encode":
        s.g = _gradients(case, seed)[0]
        s.params = B.cs_params_init(r, c, HASH_SEED, d)
        s.S = torch.zeros(r, c, **f32)
        s.wire = torch.empty(r, c, dtype=torch.int16, device=DEV)
    elif kind == "decode":
        # a path with the buffers of the aggregating side, and the tables it received
        s.path = HotPath(d, 1, r, c, k, HASH_SEED, rho=rho, device=DEV)
        acc = torch.empty(r, c, dtype=torch.int64, device=DEV)
        s.tables = []
        for g in _gradients(case, seed):
            acc.zero_()
            B.cs_fixed_accumulate(s.path.params, acc, g, 40)
            s.tables.append(torch.empty(r, c, **f32))
            B.cs_fixed_to_float(s.path.params, acc, 40, s.tables[-1])
    else:
        s.g_w = _gradients(case, seed)
        if kind == "dense":
            s.path = DenseStatePath(d, W, r, c, k, HASH_SEED, rho=rho, device=DEV, P=case["P"])
        else:
            s.path = HotPath(d, W, r, c, k, HASH_SEED, rho=rho, device=DEV, P=case["P"],
                             fold_workers=kind == "fold")
        if kind == "graph":
            s.graph = GraphedStep(s.path, s.g_w)
        if kind == "heavymix":
            s.l2sq = torch.empty(1 + r, dtype=torch.float64, device=DEV)
            s.n_heavy = torch.empty(1, dtype=torch.int64, device=DEV)
    return s


def run(s):
    if s.kind == "encode":
        B.cs_sketch_zero(s.params, s.S)
        B.cs_sketch_accumulate(s.params, s.S, s.g)
        B.cs_quantize16(s.S, s.wire, B.CS_FMT_BF16)
        return {"S": s.S, "wire": s.wire}
    p = s.path
    if s.kind == "decode":
        B.cs_sketch_merge(p.params, p.S_t, s.tables, alpha=1.0 / len(s.tables))
        p.momentum()
        p.estimate()
        p.topk()
        p.feedback()
        return {"idx": p.idx, "est": p.est, "S_u": p.S_u, "S_v": p.S_v}
    if s.kind == "heavymix":
        p.accumulate(s.g_w)
        p.merge()
        B.cs_sketch_l2sq(p.params, p.S_t, s.l2sq)
        p.estimate()
        B.cs_heavymix_select(p.est, s.k, s.l2sq, 12345, p.cand, p.est_at_cand, s.n_heavy, p.topk_ws)
        p.gather(s.g_w)
        return {"idx": p.idx, "x": p.x, "n_heavy": s.n_heavy, "l2sq": s.l2sq, "est": p.est, "S_t": p.S_t, "T": p.T}
    if s.kind == "graph":
        idx, x = s.graph.replay()
    else:
        idx, x = p.step(s.g_w)
    out = {"idx": idx, "x": x, "est": p.est, "S_t": p.S_t}
    if s.kind != "fold":
        out["T"] = p.T                                   # the workers' own tables
    if p.rho is not None:
        out["S_u"], out["S_v"] = p.S_u, p.S_v
    if s.kind == "dense":
        out["u"], out["v"] = p.u_w, p.v_w
    return out


def work(case):
    """Bytes: every vector and received table read once, every table, estimate and selection that
    the pass produces written once.  Operations: one addition per coordinate, row and worker."""
    kind, d, W, r, c, k = (case[x] for x in ("kind", "d", "W", "r", "c", "k"))
    table = 4 * r * c
    query = 4 * d + 12 * k
    if kind == "encode":
        return {"bytes": 4 * d + table + table // 2, "flops": r * d}
    state = 4 * table if case["rho"] and kind != "dense" else 0            # S_u, S_v read and written
    if kind == "decode":
        return {"bytes": W * table + state + query, "flops": r * c * W + 2 * r * d}
    read = (20 if kind == "dense" else 4) * W * d
    worker_tables = 0 if kind == "fold" else W * table
    return {"bytes": read + worker_tables + table + state + query, "flops": r * d * W + 2 * r * d}


def tolerance(case):
    """Cells are 32-bit sums of some hundred terms in an order that the hardware takes; selections
    and rounded cells may differ where two values are equal up to that."""
    return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
