"""The work that users of the bulk sampler have it do, as measurable cases.

Each case is one pass through the public entry points of `paper_2311_02909_amd.bms`, on a seeded synthetic graph
(`paper_2311_02909_amd.synth`) that stands in for a dataset:

  nodewise   sample_nodewise on a recycled result (the steady state of a training loop), every hop's arrays looked at
  ladies     sample_ladies, the same way
  forward    what follows the sampling: fetch_features of the last frontier, then aggregate_hop over every hop,
             outermost first, down to one row per seed vertex

`prepare` holds what such a program keeps: the graph on the device, the handle, the seed batches of the step, the
buffers and the result object to recycle.  The graph belongs to the case; the batches, the sampling seed and the
features to the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2311_02909_amd import bms, synth

GRAPH_SEED = 1

# the graph shapes of the repository's workloads: vertices, R-MAT pairs, quadrant weights a and b = c
TINY = dict(n=10_000, pairs=148_000, a=0.57, b=0.19)
MID = dict(n=2_450_000, pairs=94_000_000, a=0.50, b=0.17)
LARGE = dict(n=111_000_000, pairs=861_000_000, a=0.52, b=0.18)
DENSE = dict(n=8_700_000, pairs=1_280_000_000, a=0.45, b=0.22)


def _case(op, graph, k, batch, params, name=None, **options):
    case = dict(op=op, **graph, k=k, batch=batch, params=",".join(str(p) for p in params))
    case.update(options)
    if name is not None:
        case["name"] = name
    return case


def listed():
    sage = (15, 10, 5)
    return [
        # a few small minibatches of a small graph, cut apart for a training loop: launches and host work
        _case("nodewise", TINY, 4, 64, (5, 5), "tiny_sage", cut=True),
        # no bulk at all: one minibatch per call, the latency that a loop without look-ahead or a server sees
        _case("nodewise", MID, 1, 1024, sage, "one_minibatch"),
        # an ordinary bulk call on a medium graph
        _case("nodewise", MID, 64, 1024, sage, "mid_sage"),
        # the benchmark's workload: the largest graph, the most minibatches
        _case("nodewise", LARGE, 256, 1024, sage, "large_sage"),
        # long adjacency lists, the most sampled edges per call
        _case("nodewise", DENSE, 128, 1024, sage, "dense_sage"),
        # layers that also use a vertex's own features; sizes that fill no tile
        _case("nodewise", MID, 37, 1000, sage, "union_dst", variant="union_dst"),
        # independent draws
        _case("nodewise", MID, 32, 777, sage, "replace", variant="replace"),
        # wide fanouts, two layers
        _case("nodewise", MID, 8, 512, (40, 40), "wide_fanout"),
        # the layer-wise sampler with one layer and squared weights, few minibatches
        _case("ladies", MID, 3, 512, (512,), "ladies_one_layer", squared=True),
        # ... three layers, in bulk
        _case("ladies", MID, 32, 512, (512, 512, 512), "mid_ladies"),
        # ... on long adjacency lists with many samples per layer
        _case("ladies", DENSE, 64, 1024, (2048, 2048, 2048), "dense_ladies"),
        # the consumer of a bulk sample: features fetched and aggregated down to the seeds
        _case("forward", MID, 32, 1024, sage, "forward", f=100, mean=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, most_n):
    n = _log_uniform(rng, 10_000, most_n)
    degree = math.exp(rng.uniform(math.log(12.0), math.log(154.0)))
    pairs = int(min(n * degree / 2 * 1.1, 900e6))
    a = round(rng.uniform(0.45, 0.57 if n < 1_000_000 else 0.52), 3)
    b = round(rng.uniform(0.17, min(0.22, (0.97 - a) / 2)), 3)
    return dict(n=n, pairs=max(pairs, 20_000), a=a, b=b)


def draw(rng):
    op = rng.choice(["nodewise", "nodewise", "nodewise", "ladies", "ladies", "forward"])
    if op == "ladies":
        graph = _draw_graph(rng, 8_700_000)
        layers = rng.choice([1, 2, 3])
        params = [_log_uniform(rng, 64, 2048) for _ in range(layers)]
        batch = _log_uniform(rng, 64, 1024)
        # frontiers after the first are drawn in proportion to their degree: about 12 times the mean
        rows = batch + 12 * sum(params[:-1])
        most_k = 4.0e8 / (rows * (2.0 * graph["pairs"] / graph["n"]))
        k = min(_log_uniform(rng, 1, 64), max(1, int(most_k)), graph["n"] // batch)
        return _case(op, graph, k, batch, params, squared=rng.random() < 0.3)
    forward = op == "forward"
    graph = _draw_graph(rng, 8_700_000 if forward else 111_000_000)
    variant = "" if forward else rng.choice(["", "", "", "union_dst", "replace"])
    wide = not forward and rng.random() < 0.15
    if wide:
        params = [rng.randint(33, 64) for _ in range(rng.choice([1, 2]))]
    else:
        params = [rng.randint(3, 20) for _ in range(rng.choice([1, 2, 3, 3]))]
    f = _log_uniform(rng, 16, 256) if forward else 0
    most = 6.0e6 if wide else min(6.0e7, 2.0e9 / f) if forward else 8.0e7
    edges = math.exp(rng.uniform(math.log(2.0e3), math.log(most)))
    grown = float(math.prod(params))
    batch = min(_log_uniform(rng, 32, 2048), max(1, int(edges / grown)))
    k = max(1, min(int(edges / (grown * batch)), 256, graph["n"] // batch))
    if forward:
        return _case(op, graph, k, batch, params, f=f, mean=rng.random() < 0.5)
    case = _case(op, graph, k, batch, params, cut=k * len(params) <= 12 and rng.random() < 0.5)
    if variant:
        case["variant"] = variant
    return case


@functools.lru_cache(maxsize=4)
def _graph(n, pairs, a, b):
    return synth.rmat_graph(n=n, pairs=pairs, a=a, b=b, c=b, seed=GRAPH_SEED, device="cuda")


def _graph_of(case):
    return _graph(case["n"], case["pairs"], case["a"], case["b"])


# The sizes of a sample depend on the draws.  A program that wants arrays of one shape whatever was drawn (to capture
# its training step in a graph, say) gives the library buffers of its own, with room to spare, and uses them whole.
SPARE = 1 << 18


class _Pool(bms.TorchAllocator):
    """Zeroed buffers with spare room for a result (bms_opts.alloc), found again by the address of an array."""

    def __init__(self):
        super().__init__("cuda")

        def alloc(nbytes, _ctx):
            try:
                t = torch.zeros(4 * int(nbytes) + 16 * SPARE, dtype=torch.uint8, device="cuda")
            except RuntimeError:
                return None
            self.live[t.data_ptr()] = t
            return t.data_ptr()

        def dealloc(ptr, _ctx):
            self.live.pop(ptr, None)
            self.arrays.clear()

        self.alloc, self.dealloc = bms.ALLOC_FN(alloc), bms.DEALLOC_FN(dealloc)
        self.arrays = {}

    def whole(self, view, room):
        """The first `room` elements of the buffer that `view` starts."""
        if view is None:
            return None
        if view.numel() > room:
            raise ValueError("an array of %d elements does not fit the %d provided" % (view.numel(), room))
        if view.numel() == 0:
            return torch.zeros(room, dtype=view.dtype, device="cuda")
        key = (view.data_ptr(), view.dtype, room)
        whole = self.arrays.get(key)
        if whole is None:
            buffer = self.live[view.data_ptr()]
            whole = buffer[:buffer.numel() // 8 * 8].view(view.dtype)[:room]
            if whole.numel() < room:
                raise ValueError("a buffer of %d elements is smaller than the %d provided" % (whole.numel(), room))
            self.arrays[key] = whole
        return whole


def _params(case):
    return [int(p) for p in case["params"].split(",")]


def _sample(case, csr, batches, seed, result=None, pool=None):
    if case["op"] == "ladies":
        return bms.sample_ladies(csr, batches, _params(case), seed, squared=case.get("squared", False), recycle=result,
                                 allocator=pool)
    variant = case.get("variant", "")
    return bms.sample_nodewise(csr, batches, _params(case), seed, union_dst=variant == "union_dst",
                               replace=variant == "replace", recycle=result, allocator=pool)


@functools.lru_cache(maxsize=32)
def _pilot(items):
    """Sizes of one sampling call of the case, per hop: rows, nnz, ncols, pnnz, neighbours of the rows; and the
    distinct vertices of the last frontier."""
    case = dict(items)
    g = _graph_of(case)
    csr = bms.Csr(g.rowptr, g.col)
    batches = synth.train_batches(g.n, 1.0, case["k"], case["batch"], 1, device="cuda")
    hops = _sample(case, csr, batches, 42).hops()
    sizes = []
    for h in hops:
        rows = h.row_vertex.long()
        sizes.append((h.rows, h.nnz, h.ncols, h.pnnz, int((g.rowptr[rows + 1] - g.rowptr[rows]).sum())))
    return sizes, int(torch.unique(hops[-1].col_vertex).numel())


def _sizes(case):
    return _pilot(tuple(sorted((key, v) for key, v in case.items() if key != "name")))


def prepare(case, seed):
    g = _graph_of(case)
    room = [[2 * x + SPARE for x in hop] for hop in _sizes(case)[0]]
    state = dict(case=case, csr=bms.Csr(g.rowptr, g.col), seed=seed * 2654435761 + 42, room=room, pool=_Pool(), result=None,
                 batches=synth.train_batches(g.n, 1.0, case["k"], case["batch"], seed, device="cuda"))
    if case["op"] == "forward":
        state["result"] = _sample(case, state["csr"], state["batches"], state["seed"])
        generator = torch.Generator(device="cuda").manual_seed(seed)
        state["H"] = torch.randn((g.n, case["f"]), dtype=torch.float32, device="cuda", generator=generator)
        state["X"] = [torch.zeros((room[-1][2], case["f"]), dtype=torch.float32, device="cuda")]
        state["X"] += [torch.zeros((rows, case["f"]), dtype=torch.float32, device="cuda") for rows, *_ in reversed(room)]
    return state


def run(state):
    case = state["case"]
    if case["op"] == "forward":
        result, X = state["result"], state["X"]
        hops = result.sizes()
        _, _, columns = hops[-1]
        x = bms.fetch_features(state["H"], result.hop(len(hops) - 1).col_vertex, out=X[0][:columns])
        for out, h in zip(X[1:], range(len(hops) - 1, -1, -1)):
            x = bms.aggregate_hop(result, h, x, mean=case["mean"], out=out[:hops[h][0]])
        return X
    pool, room = state["pool"], state["room"]
    result = state["result"] = _sample(case, state["csr"], state["batches"], state["seed"], state["result"], pool)
    if case.get("cut", False):
        # as a training loop goes over them: every minibatch with its own sampled adjacency of every hop
        cut = [[result.minibatch(h, i) for h in range(len(room))] for i in range(case["k"])]
        parts = [[m.row0, m.edge0, m.col0, m.rows, m.nnz, m.ncols, m.row_vertex.numel(), m.rowptr.numel(), m.col.numel(),
                  m.col_vertex.numel()] for hops in cut for m in hops]
        first = [[pool.whole(m.row_vertex, r[0]), pool.whole(m.rowptr, r[0]), pool.whole(m.col, r[1]),
                  pool.whole(m.col_vertex, r[2]), pool.whole(m.row_self, r[0])] for m, r in zip(cut[0], room)]
        return [np.array(parts), first]
    return [[h.rows, h.nnz, h.ncols, h.pnnz, h.mb_rowoff, h.mb_coloff, h.p_off, pool.whole(h.row_vertex, r[0]),
             pool.whole(h.rowptr, r[0]), pool.whole(h.col, r[1]), pool.whole(h.col_vertex, r[2]), pool.whole(h.p_col, r[3]),
             pool.whole(h.p_cnt, r[3]), pool.whole(h.row_self, r[0])] for h, r in zip(result.hops(), room)]


def work(case):
    """Bytes of one pass, from the sizes that one sampling call of the case gives.

    nodewise, per hop of R rows, E sampled edges, U columns: row extents 16 R, sampled neighbours 4 E, rowptr 8 R,
    col 4 E, col_vertex 4 U.  ladies: the rows' D neighbours 4 D instead of the sampled ones, and P (8 bytes per
    entry).  forward: the fetched rows of H once and written once, per hop the columns' rows read once, the CSR, and
    the output; one addition per edge and feature.
    """
    hops, distinct = _sizes(case)
    if case["op"] == "forward":
        f = case["f"]
        moved = hops[-1][2] * (4 + 4 * f) + distinct * 4 * f
        moved += sum(4 * nnz + 8 * rows + 4 * f * (ncols + rows) for rows, nnz, ncols, _, _ in hops)
        return {"bytes": moved, "flops": f * sum(hop[1] for hop in hops)}
    moved = 4 * case["k"] * case["batch"]
    for rows, nnz, ncols, pnnz, gathered in hops:
        moved += 24 * rows + 4 * nnz + 4 * ncols
        moved += 4 * gathered + 8 * pnnz if case["op"] == "ladies" else 4 * nnz
    return {"bytes": moved, "flops": 0}


def tolerance(case):
    # the samplers return whole numbers; the aggregation adds up to a few dozen fp32 values per output
    return {"rel": 1e-5} if case["op"] == "forward" else "exact"
