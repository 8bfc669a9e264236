"""One pass of the hot path on one GPU: buffers and the order of library calls, nothing else.

Per step (Alg. 3 of the paper, with the W workers simulated on the one device):
    worker sketches   S^w = S(g^w)                cs_bundle_sketch  (T[w/8][j][b][w%8]), with the next two steps; where
                                                  the sketch has no lists cs_sketch_accumulate_bundle
    aggregate         S_t = (1/W) sum_w S^w       cs_bundle_merge[_momentum]
                      (fold_workers: S_t = S((1/W) sum_w g^w), cs_vectors_sum, cs_sketch_accumulate)
    momentum, error   S_u = rho S_u + S_t ; S_v += S_u      cs_sketch_momentum   (stateful only)
    query all         est = estimate(S_v or S_t)  cs_sketch_estimate
    choose largest    idx = top-k |est|           cs_heavy_hitters_topk_kept
    second round      x = (1/W) sum_w g^w[idx]    cs_gather_exact
    feedback          S_v -= S(est[idx]) ; S_u -= S(estimate(S_u, idx))   cs_sketch_feedback_pair (stateful)
step queries and chooses in one launch for short vectors (cs_sketch_estimate_topk), and second
round and feedback together (cs_gather_feedback).  Update of short vectors: cs_bundle_sketch_lists.
Every arithmetic step runs inside libcsketch.so; this class only owns tensors (and counts `hist` of
short vectors for whoever asks).
"""
from __future__ import annotations

import ctypes

import torch

from . import binding as B


class HotPath:
    # the update by way of running sums (cs_bundle_sketch), where the sketch has lists for it: its index, its
    # workspace, and what they were made for: the sketch's parameters, fold_workers, W and d
    _index = _sums_ws = _sums_params = _sums_for = None
    _cell_lists = False                  # _index holds cell lists (cs_bundle_sketch_lists): short vectors
    SUMS_OWN_BYTES = 2 << 30             # the workspace, or the cell lists: up to here, else the path does without (0: in any case)

    def __init__(self, d: int, W: int, r: int, c: int, k: int, seed: int,
                 rho: float | None = None, device="cuda:0", P: int = 1, fold_workers: bool = False):
        """P > 1: the sketch is queried for the top P*k coordinates, the workers for their exact
        values, and the k largest exact sums are kept (Alg. 3 as the paper trains with it).
        fold_workers: the workers, which share this GPU, are summed before they are sketched
        (every vector is read once; the sum goes into d floats of scratch, then straight into
        S_t; of short vectors each coordinate's sum is taken where a cell needs it, r times): no
        worker tables, no merge.  The scratch is the query's, so the stages of one
        path run one after the other; where the query has none (short vectors and column counts
        without a traversal plan) the path holds d floats more.
        Memory beside the tables and est: the query's scratch (r d floats for long vectors), for short
        vectors the lists of the cells' coordinates (r (c + d) words, 1.3 MB at d = 65 536, 5 x 1024; up to
        240 MB, for the sum of folded vectors of 4 million and 15 rows of a few columns), and where the
        update goes by way of running sums (up to 4 workers, up to 16 with short vectors, up to 64 with
        vectors of 32 million on) their index and workspace, 35 MB at d = 6.5 M, W = 4, 5 x 2^17 and 1.9 GB
        at d = 10^8, W = 32, 5 x 2^20, where they save 1.8 % of the update: SUMS_OWN_BYTES, of the class or a
        subclass, bounds the workspace and the lists."""
        self.d, self.W, self.r, self.c, self.k = d, W, r, c, k
        self.P = P
        self.fold_workers = fold_workers
        self.kq = min(P * k, d)          # coordinates asked of the sketch
        self.rho = rho
        self.device = torch.device(device)
        self.params = B.cs_params_init(r, c, seed, d)
        f32 = dict(dtype=torch.float32, device=self.device)
        # the W workers' sketches as one bundle: T[w // 8][j][b][w % 8] = S^w[j][b]
        self.T = torch.zeros(B.cs_bundle_floats(self.params, 1 if fold_workers else W), **f32)
        self.S_t = torch.zeros(r, c, **f32)
        self.S_u = torch.zeros(r, c, **f32) if rho is not None else None
        self.S_v = torch.zeros(r, c, **f32) if rho is not None else None
        self.est = torch.empty(d, **f32)
        self.cand = torch.empty(self.kq, dtype=torch.int64, device=self.device)
        self.est_at_cand = torch.empty(self.kq, **f32)
        self.x_cand = torch.empty(self.kq, **f32)
        # with P = 1 the candidates are the selection
        self.idx = self.cand if P == 1 else torch.empty(k, dtype=torch.int64, device=self.device)
        self.est_at_idx = self.est_at_cand
        self.x = self.x_cand if P == 1 else torch.empty(k, **f32)
        self.delta = torch.empty(k, **f32)
        self.uhat = torch.empty(k, **f32)
        self.topk_ws = torch.empty(B.cs_topk_workspace_bytes(d, self.kq), dtype=torch.uint8,
                                   device=self.device)
        B.cs_topk_workspace_clear(self.topk_ws)      # once: every selection leaves it clear
        self._counts = torch.zeros(B.CS_TOPK_HIST_BINS, dtype=torch.int64, device=self.device)
        n_est = B.cs_estimate_scratch_bytes(self.params, d)
        self.est_ws = (torch.empty(n_est, dtype=torch.uint8, device=self.device)
                       if n_est else None)
        self.g_mean = None
        if fold_workers and W > 1:
            self._mean_buffer(d)
        if not self._build_cell_lists():
            self._build_index()

    # individual stages (bench.py times them separately) ---------------------------------
    def worker_table(self, w: int):
        """Worker w's own sketch (a strided view of the bundle)."""
        g = B.CS_BUNDLE_GROUP
        return self.T.view(-1, self.r, self.c, g)[w // g, :, :, w % g]

    def _mean_buffer(self, n: int):
        """n floats for the mean of folded workers: the query's scratch, which is free until the
        estimate, or memory that is kept where the query needs too little of it"""
        if self.g_mean is None or self.g_mean.numel() < n:
            size = max(n, self.d)
            fits = self.est_ws is not None and self.est_ws.numel() >= 4 * size
            self.g_mean = (self.est_ws[:4 * size].view(torch.float32) if fits
                           else torch.empty(size, dtype=torch.float32, device=self.device))
        return self.g_mean[:n]

    def _build_cell_lists(self):
        """for short vectors; True where there are some"""
        n = B.cs_cell_lists_bytes(self.params, 0 if self.fold_workers else self.W, self.d)
        if not n or n > self.SUMS_OWN_BYTES:
            return False
        self._index = torch.empty(n, dtype=torch.uint8, device=self.device)
        B.cs_cell_lists_build(self.params, self.d, self._index)
        self._cell_lists = True
        # folded workers: all of them cell by cell while that is less than a launch more, else their sum
        self._sum_first = self.W > 1 and (self.r * self.d * self.W > 1_250_000 or self.W > 256)
        self._sums_params = self._lists()
        self._sums_for = self.fold_workers, self.W, self.d
        return True

    def _build_index(self):
        n = B.cs_update_index_bytes(self.params, 0 if self.fold_workers else self.W, self.d)
        if not n:
            return
        W = 1 if self.fold_workers else self.W
        need = B.cs_update_workspace_bytes(self.params, W, self.d)
        if need > self.SUMS_OWN_BYTES:
            return
        # (memory of its own, not the query's scratch: accumulate alone, workers not folded, may run beside the query
        # of the step before; folded workers' mean lies in that scratch, and the later stages write what the query reads)
        self._sums_ws = torch.empty(need, dtype=torch.uint8, device=self.device)
        self._index = torch.empty(n, dtype=torch.uint8, device=self.device)
        B.cs_update_index_build(self.params, self.d, self._index)
        self._sums_params = self._lists()
        self._sums_for = self.fold_workers, W, self.d

    def _lists(self):
        """the parameters as they are now, byte for byte, up to the visit lists of the last row (what lies behind are
        lists that neither the index, which is for powers of two, nor the cell lists depend on)"""
        n = B.CsParams.visit.offset + self.r * ctypes.sizeof(B.CsVisitPlan)
        return memoryview(self.params).cast("B")[:n].tobytes()

    def _indexed(self, g_w):
        """The vectors and the sketch are those that the index and its workspace were made for.  (Whoever gives a path
        another sketch may do so by replacing its parameters or in place.)"""
        if self._index is None:
            return False
        fold, W, d = self._sums_for
        return (self.fold_workers == fold and (len(g_w) == W or fold and not self._cell_lists) and g_w[0].numel() == d
                and self._lists() == self._sums_params)

    def _mean(self, g_w):
        """the mean of folded workers, in scratch"""
        n = g_w[0].numel()
        mean = self.g_mean
        if mean is None or mean.numel() != n:
            mean = self._mean_buffer(n)
        B.cs_vectors_sum(g_w, mean, alpha=1.0 / self.W)
        return mean

    def _sketch_indexed(self, g_w, **tables):
        """accumulate, and with the tables S_t (S_u, S_v) what follows it, in the pass that gathers the sums"""
        if self._cell_lists:
            T, alpha = self.T, 1.0 / self.W
            if self.fold_workers:
                T, tables = None, {"S_t": self.S_t, **tables}
                if self._sum_first:
                    g_w, alpha = [self._mean(g_w)], 1.0
            B.cs_bundle_sketch_lists(self.params, T, g_w, self._index, alpha=alpha, **tables)
            return
        if not self.fold_workers:
            B.cs_bundle_sketch(self.params, self.T, g_w, self._index, self._sums_ws, alpha=1.0 / self.W, **tables)
        elif len(g_w) == 1:
            B.cs_bundle_sketch(self.params, None, g_w, self._index, self._sums_ws, 1.0 / self.W,
                               **{"S_t": self.S_t, **tables})
        else:
            B.cs_bundle_sketch(self.params, None, [self._mean(g_w)], self._index, self._sums_ws,
                               **{"S_t": self.S_t, **tables})

    def accumulate(self, g_w):
        if self._indexed(g_w):
            self._sketch_indexed(g_w)
            return
        if self.fold_workers:
            B.cs_sketch_zero(self.params, self.S_t)
            if len(g_w) == 1:
                B.cs_sketch_accumulate(self.params, self.S_t, g_w[0], scale=1.0 / self.W)
            else:
                B.cs_sketch_accumulate(self.params, self.S_t, self._mean(g_w))
            return
        B.cs_bundle_zero(self.params, self.T, self.W)
        B.cs_sketch_accumulate_bundle(self.params, self.T, g_w)

    def merge(self):
        if self.fold_workers:
            return                       # S_t is complete already
        B.cs_bundle_merge(self.params, self.S_t, self.T, self.W, alpha=1.0 / self.W, beta=0.0)

    def momentum(self):
        if self.rho is not None:
            B.cs_sketch_momentum(self.params, self.S_u, self.S_v, self.S_t, self.rho)

    def query_table(self):
        return self.S_v if self.rho is not None else self.S_t

    @property
    def hist(self):
        """Counts of est by magnitude bin.  The estimate fills them where the selection reads them;
        up to CS_TOPK_SMALL_D coordinates, whose selection counts by itself, they are taken here,
        so that a step does not launch for them."""
        if self.d <= B.CS_TOPK_SMALL_D:
            bins = ((self.est.view(torch.int32) & 0x7FFFFFFF) >> 20).long()
            self._counts.zero_().scatter_add_(0, bins, torch.ones_like(bins))
        return self._counts

    @hist.setter
    def hist(self, counts):
        self._counts = counts

    def _hist(self):
        """the counts, where the selection reads them"""
        return self._counts if self.d > B.CS_TOPK_SMALL_D else None

    def estimate(self):
        B.cs_sketch_estimate(self.params, self.query_table(), self.est, 0, self.est_ws, self._hist())

    def topk(self):
        B.cs_heavy_hitters_topk_kept(self.est, self.kq, self.cand, self.est_at_cand, self.topk_ws, self._hist())

    def gather(self, g_w):
        B.cs_gather_exact(g_w, self.cand, self.x_cand, alpha=1.0 / self.W)
        if self.P > 1:
            B.cs_select_exact_topk(self.cand, self.x_cand, self.k, self.idx, self.x, self.topk_ws)

    def feedback(self):
        if self.rho is not None:
            B.cs_sketch_feedback_pair(self.params, self.S_v, self.S_u, self.idx, self.delta, self.uhat)

    def aggregate(self):
        """merge and momentum, in one pass where the workers have tables of their own and neither
        stage is overridden"""
        cls, own = type(self), self.__dict__
        if (self.rho is None or self.fold_workers
                or cls.merge is not HotPath.merge or cls.momentum is not HotPath.momentum
                or "merge" in own or "momentum" in own):
            self.merge()
            self.momentum()
            return
        B.cs_bundle_merge_momentum(self.params, self.S_t, self.S_u, self.S_v, self.T, self.W, 1.0 / self.W, self.rho)

    def _not_overridden(self, *stages):
        cls, own = type(self), self.__dict__
        for x in stages:
            if x in own or (cls is not HotPath and getattr(cls, x) is not getattr(HotPath, x)):
                return False
        return True

    def sketch_and_aggregate(self, g_w):
        """accumulate, merge and momentum: the last two come out of the pass that writes the tables, where there
        is one and no stage is overridden"""
        if self._indexed(g_w) and self._not_overridden("accumulate", "merge", "momentum", "aggregate"):
            state = {} if self.rho is None else {"S_u": self.S_u, "S_v": self.S_v, "rho": self.rho}
            self._sketch_indexed(g_w, S_t=self.S_t, **state)
            return
        self.accumulate(g_w)
        self.aggregate()

    def query_and_choose(self):
        """estimate and topk, in one launch for short vectors"""
        short = B.CS_QUERY_CHOOSE_CELLS
        if (self.r * self.d <= short and self.params.r * self.est.numel() <= short    # (the sketch may have been replaced)
                and self._not_overridden("estimate", "topk")):
            B.cs_sketch_estimate_topk(self.params, self.query_table(), self.est, self.kq, self.cand, self.est_at_cand)
            return
        self.estimate()
        self.topk()

    def second_round(self, g_w):
        """gather and feedback, which share a launch where both begin with the candidates"""
        if self.rho is not None and self.P == 1 and self.idx is self.cand and self._not_overridden("gather", "feedback"):
            B.cs_gather_feedback(self.params, g_w, self.cand, self.x_cand, self.S_v, self.S_u, self.delta, self.uhat,
                                 alpha=1.0 / self.W)
            return
        self.gather(g_w)
        self.feedback()

    def step(self, g_w):
        """g_w: list of W fp32[d] device tensors.  Returns (idx, x): chosen coordinates
        (ascending) and their exact mean over workers."""
        g_w = B.DeviceVectors(g_w, name="g_w")
        self.sketch_and_aggregate(g_w)
        self.query_and_choose()
        self.second_round(g_w)
        return self.idx, self.x


class ReproduciblePath(HotPath):
    """The same step with sums that do not depend on the order of the additions, for debugging
    and for checkpoints that must resume bit for bit: the workers' vectors and the feedback go
    through the 64-bit fixed-point update (every contribution rounded once to a multiple of
    2^-frac_bits, integer sums), everything else is elementwise or integer already.  Two runs on
    equal inputs give equal bits; about one atomic request per coordinate and row, so far
    slower than HotPath.

        worker sketches   acc += fixed(g^w) for every w            cs_fixed_accumulate
        aggregate         S_t = float(acc) / W                     cs_fixed_to_float
        feedback          val = estimate(S, idx); S += float(fixed(-val at idx))
                          cs_sketch_estimate_sparse, cs_fixed_accumulate_sparse, cs_sketch_axpby
    `dropped` counts the coordinates that were left out (not finite, or too large for the
    chosen frac_bits) since the object was made."""

    def _build_cell_lists(self):
        return False                                  # (its update is another)

    def _build_index(self):
        pass

    def __init__(self, d, W, r, c, k, seed, rho=None, device="cuda:0", frac_bits: int = 40):
        super().__init__(d, 1, r, c, k, seed, rho=rho, device=device)     # no bundle of W tables
        self.W = W
        self.frac_bits = frac_bits
        self.acc = torch.zeros(r, c, dtype=torch.int64, device=self.device)
        self.dropped = torch.zeros(1, dtype=torch.int64, device=self.device)
        self.S_fb = torch.empty(r, c, dtype=torch.float32, device=self.device)

    def accumulate(self, g_w):
        self.acc.zero_()
        for g in g_w:
            B.cs_fixed_accumulate(self.params, self.acc, g, self.frac_bits, dropped=self.dropped)

    def merge(self):
        B.cs_fixed_to_float(self.params, self.acc, self.frac_bits, self.S_t, alpha=1.0 / self.W)

    def _feedback(self, S, val):
        B.cs_sketch_estimate_sparse(self.params, S, self.idx, val)
        self.acc.zero_()
        B.cs_fixed_accumulate_sparse(self.params, self.acc, self.idx, val, self.frac_bits,
                                     scale=-1.0, dropped=self.dropped)
        B.cs_fixed_to_float(self.params, self.acc, self.frac_bits, self.S_fb)
        B.cs_sketch_axpby(self.params, S, 1.0, self.S_fb, 1.0)

    def feedback(self):
        if self.rho is not None:
            self._feedback(self.S_v, self.delta)
            self._feedback(self.S_u, self.uhat)


class DenseStatePath(HotPath):
    """Alg. 3 as printed: momentum u^w and error accumulation v^w are dense vectors on every
    worker (2 W d floats), the sketch is taken of v^w, the second round returns exact sums of
    v^w, and u^w, v^w are zeroed on the coordinates of the update.  Costs one more streaming
    pass over the state (20 bytes per coordinate and worker) than the sketch-space form.

        momentum, error   u^w = rho u^w + g^w ; v^w += u^w          cs_dense_momentum
        worker sketches   S^w = S(v^w)                              cs_sketch_accumulate_bundle
        aggregate, query, choose                                    as in HotPath (stateless)
        second round      x = (1/W) sum_w v^w[idx]                  cs_gather_exact
        masking           u^w[idx] = v^w[idx] = 0                   cs_dense_mask
    """

    def __init__(self, d, W, r, c, k, seed, rho, device="cuda:0", P: int = 1):
        super().__init__(d, W, r, c, k, seed, rho=None, device=device, P=P)
        self.m = rho
        f32 = dict(dtype=torch.float32, device=self.device)
        self.u_w = [torch.zeros(d, **f32) for _ in range(W)]
        self.v_w = [torch.zeros(d, **f32) for _ in range(W)]

    def dense_momentum(self, g_w):
        B.cs_dense_momentum(self.u_w, self.v_w, g_w, self.m)

    def mask(self):
        B.cs_dense_mask(self.u_w, self.v_w, self.idx)

    def step(self, g_w):
        self.dense_momentum(g_w)
        if self._indexed(self.v_w) and self._not_overridden("accumulate", "merge"):
            self._sketch_indexed(self.v_w, S_t=self.S_t)
        else:
            self.accumulate(self.v_w)
            self.merge()
        self.query_and_choose()
        self.gather(self.v_w)
        self.mask()
        return self.idx, self.x


class GraphedStep:
    """One step of a HotPath (or DenseStatePath) captured once as a HIP graph and replayed.

    Every stage of a step is a fixed sequence of kernel launches on the caller's stream with
    fixed device pointers -- no allocation, no host synchronisation, no memset node -- so the
    whole step can be recorded and replayed with one submission.  That pays where the host is what a
    step waits for: where the program waits for every step (us per step, eager / replayed, 4 workers with momentum), d = 784:
    43 / 39, d = 30 403: 64 / 58, d = 2^20: 116 / 111.  Steps enqueued one behind the other run ahead of the device, and then
    the kernels of a graph follow each other a little more slowly than those of a stream: d = 784: 27 / 27, d = 30 403:
    42 / 46, d = 2^20: 94 / 98, d = 6.5 M: 347 / 351.  The gradients live in static buffers `g_w` that the
    caller overwrites before each replay; results appear in the HotPath's own tensors."""

    def __init__(self, path: HotPath, g_w):
        self.path = path
        self.g_w = g_w
        # one warm-up step outside the capture, on a side stream (a captured launch does not
        # execute, the warm-up does: the state it advanced is put back afterwards)
        saved = [t.clone() for t in self._state()]
        side = torch.cuda.Stream(device=path.device)
        side.wait_stream(torch.cuda.current_stream(path.device))
        with torch.cuda.stream(side):
            path.step(g_w)
        torch.cuda.current_stream(path.device).wait_stream(side)
        torch.cuda.synchronize(path.device)
        for t, s in zip(self._state(), saved):
            t.copy_(s)
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            path.step(g_w)

    def _state(self):
        p = self.path
        out = [t for t in (p.S_u, p.S_v) if t is not None]
        out += list(getattr(p, "u_w", [])) + list(getattr(p, "v_w", []))
        return out

    def replay(self):
        self.graph.replay()
        return self.path.idx, self.path.x
