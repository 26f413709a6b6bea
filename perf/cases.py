"""What the performance of this library is measured on: mini-batches of the benchmark's graphs through the public entry
points (sampling + retrieve as one unit, as two calls, sampling alone, the neighbour mean behind it, a FIFO-cached step,
an explicit gather, a pipeline), from the smallest calls to the largest, and cases drawn from the same ranges.

A graph and its feature rows are what a training program loads once and keeps for every mini-batch, so they are made once
per process (from the configuration's own graph seed); the seed given to prepare() decides the mini-batch: the seed nodes,
the sampling seed, the ids of an explicit gather.
"""
import math

import numpy as np
import torch

import paper_2511_07421_amd as a3
from workloads import get_config, make_graph, seed_batch

_LINE = 128                       # padded rows start a whole number of cache lines apart
_A = 2.1                          # exponent of the graphs' degree law

# path: which entry points a pass goes through
#   unit      sample_gather_begin, sample_blocks_end
#   split     sample_blocks_begin, gather_input_features, sample_blocks_end
#   mean      unit, then the neighbour mean of the outermost block, queued before the host knows any count
#   sample    sample_blocks
#   fifo      unit, then the FIFO cache's update with the rows just retrieved
#   ids       gather_features for a list of ids
#   pipeline  six mini-batches through a parallel pipeline of three workers (mode 1)
_LISTED = [
    # the smallest training mini-batch that the repository configures: launches and latency are all there is
    dict(name="tiny_unit", path="unit", graph="tiny", batch=256, fanouts="10,5", cache=1.0, gamma=1.0, padded=False),
    # a request for a few nodes, three hops, four fifths of the feature rows in host memory, biased to cached nodes
    dict(name="request_16", path="split", graph="copurchase", batch=16, fanouts="15,10,5", cache=0.2, gamma=4.0, padded=True),
    # the dense social graph's training mini-batch with the first aggregation of its forward pass, rows padded
    dict(name="social_mean", path="mean", graph="social", batch=1024, fanouts="25,10", cache=1.0, gamma=1.0, padded=True),
    # the same graph with the paper's second fanout pair, packed rows and an odd batch (the last of an epoch)
    dict(name="social_packed_odd", path="split", graph="social", batch=509, fanouts="25,15", cache=1.0, gamma=1.0, padded=False),
    # the paper's setting: a partly cached table, sampling biased to the cached nodes, misses over the host link
    dict(name="copurchase_biased", path="unit", graph="copurchase", batch=4096, fanouts="15,10,5", cache=0.2, gamma=4.0, padded=True),
    # biased sampling by itself (the caller retrieves elsewhere)
    dict(name="copurchase_sampling", path="sample", graph="copurchase", batch=4096, fanouts="15,10,5", cache=0.5, gamma=2.0, padded=True),
    # the largest batch of the benchmark's sweep with everything in device memory
    dict(name="copurchase_16k", path="unit", graph="copurchase", batch=16384, fanouts="15,10,5", cache=1.0, gamma=1.0, padded=True),
    # the headline: 100 M nodes, 8-byte ids, half-precision rows
    dict(name="citation_step", path="unit", graph="citation", batch=8192, fanouts="15,10,5", cache=1.0, gamma=1.0, padded=True),
    # one wide hop from many nodes of that graph, as layer-wise inference asks for it
    dict(name="citation_one_hop", path="split", graph="citation", batch=30011, fanouts="50", cache=1.0, gamma=1.0, padded=True),
    # a dynamic cache: the mini-batch's misses enter the FIFO ring behind the retrieve
    dict(name="fifo_step", path="fifo", graph="copurchase", batch=4096, fanouts="15,10,5", cache=0.2, gamma=4.0, padded=False),
    # rows of a caller's own id list, row number = id, no device map
    dict(name="gather_ids", path="ids", graph="citation", batch=700001, fanouts="", cache=1.0, gamma=1.0, padded=True),
    # mini-batches in flight on three streams, as a training loop keeps them
    dict(name="social_pipeline", path="pipeline", graph="social", batch=1024, fanouts="25,10", cache=1.0, gamma=1.0, padded=True),
]
_PIPE_BATCHES, _PIPE_WORKERS = 6, 3
_FIFO_BATCHES = 16                # seed batches that a FIFO state goes through in turn


def listed():
    return [dict(c) for c in _LISTED]


# ---- sizes ---------------------------------------------------------------------------------------------------------
_LAWS = {}


def _law(graph):
    """(nodes per class, degree) of a graph's degree law, in classes that thin out towards the hubs"""
    if graph not in _LAWS:
        w = get_config(graph)
        edge = np.exp(-np.linspace(0.0, math.log(w.num_nodes), 2001))   # share of nodes above a class
        nodes = -np.diff(np.append(edge, 0.0)) * w.num_nodes
        shape = np.append(np.sqrt(edge[:-1] * edge[1:]), edge[-1]) ** (-1.0 / (_A - 1.0))
        lo, hi = 1e-3, float(w.d_max)
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            mean = (nodes * np.clip(mid * shape, w.d_min, w.d_max)).sum() / w.num_nodes
            lo, hi = (mid, hi) if mean < w.mean_degree else (lo, mid)
        _LAWS[graph] = nodes, np.clip(hi * shape, w.d_min, w.d_max)
    return _LAWS[graph]


def _fanouts(case):
    return [int(f) for f in str(case["fanouts"]).split(",") if f]


def _expected(case):
    """Expected sizes of a mini-batch: destinations and edges per hop, input nodes, input nodes not cached.  Mean field:
    every node of a degree class is in the frontier with the same probability, neighbours are met in proportion to their
    degree (as the generator draws them), cached ones gamma times as often."""
    nodes, deg = _law(case["graph"])
    cached = np.cumsum(nodes[::-1])[::-1] <= case["cache"] * nodes.sum() * (1 + 1e-9)
    pull = deg * np.where(cached, case["gamma"] if case["path"] != "ids" else 1.0, 1.0)
    pull = pull / (nodes * pull).sum()
    inside = np.full(len(nodes), min(1.0, case["batch"] / nodes.sum()))
    dst, edges = [], []
    for f in _fanouts(case):
        dst.append(float((nodes * inside).sum()))
        edges.append(float((nodes * inside * np.minimum(deg, f)).sum()))
        inside = 1.0 - (1.0 - inside) * np.exp(-edges[-1] * pull)
    return dst, edges, float((nodes * inside).sum()), float((nodes * inside * ~cached).sum())


def _row_bytes(case):
    return get_config(case["graph"]).row_bytes


def work(case):
    """ids, row bounds and chosen neighbours read once; blocks, input nodes and rows written once; rows read once"""
    w = get_config(case["graph"])
    ib, row = torch.empty(0, dtype=w.idx_dtype).element_size(), w.row_bytes
    if case["path"] == "ids":
        return {"bytes": case["batch"] * (ib + 2.0 * row), "flops": 0.0}
    dst, edges, n_in, n_host = _expected(case)
    total = sum(dst) * (ib + 16 + 4) + sum(edges) * (ib + 4 + 8) + n_in * ib
    flops = 0.0
    if case["path"] != "sample":
        total += n_in * (4 + 2.0 * row)
    if case["path"] == "mean":
        total += n_in * row + dst[-1] * row
        flops += edges[-1] * w.feat_dim
    if case["path"] == "fifo":
        total += n_host * (2.0 * row + 12)
    if case["path"] == "pipeline":
        total *= _PIPE_BATCHES
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """Ids, offsets and copied rows have one right answer.  The mean is a 32-bit sum of at most thirty terms: against sums in
    64 bits it is off by 1.1e-7 of its norm and 8e-7 at its worst element; rounded to half precision, one sum in some
    thousands falls on the other side of a rounding step, 1e-3 of its value."""
    if case["path"] != "mean":
        return "exact"
    return {"rel": 4e-7, "max": 3e-6} if get_config(case["graph"]).feat_dtype == torch.float32 else {"rel": 1e-4, "max": 2e-3}


_MOST_BYTES, _MOST_HOST_BYTES, _MOST_EDGES, _MOST_BOUND = 750e6, 60e6, 2.3e6, 18e6


def _fits(case):
    """no drawn case costs more than the largest listed ones"""
    if case["path"] == "ids":
        return True
    dst, edges, n_in, n_host = _expected(case)
    fan = _fanouts(case)
    times = _PIPE_BATCHES if case["path"] == "pipeline" else 1
    bound = case["batch"] * math.prod(1 + f for f in fan)
    limit = _MOST_BYTES * (4 if times > 1 else 1)
    return (work(case)["bytes"] <= limit and n_host * _row_bytes(case) <= _MOST_HOST_BYTES and sum(edges) * times <= _MOST_EDGES
            and bound <= _MOST_BOUND)


def draw(rng):
    spans = {"tiny": (8, 2048), "social": (8, 1500), "copurchase": (8, 16384), "citation": (8, 12000)}
    while True:
        path = rng.choice(["unit", "unit", "split", "mean", "sample", "sample", "fifo", "ids", "pipeline"])
        if path == "ids":
            graph = rng.choice(["social", "copurchase", "citation"])
            top = min(700000, int(180e6 / get_config(graph).row_bytes))
            batch, fanouts = int(round(math.exp(rng.uniform(math.log(1000), math.log(top))))), ""
        else:
            graph = rng.choice({"fifo": ["copurchase"], "mean": ["tiny", "social", "copurchase", "citation"],
                                "pipeline": ["tiny", "social", "copurchase"]}.get(path, ["tiny", "social", "copurchase", "copurchase", "citation"]))
            low, high = spans[graph]
            batch = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
            hops = rng.choice([1, 2, 2, 3, 3])
            fanouts = ",".join(str(int(round(math.exp(rng.uniform(math.log(3), math.log(30)))))) for _ in range(hops))
        partly = graph == "copurchase" and path not in ("ids", "pipeline")
        cache = round(rng.uniform(0.05, 0.6), 3) if partly and (path == "fifo" or rng.random() < 0.6) else 1.0
        gamma = rng.choice([1.0, 1.5, 2.0, 4.0, 8.0]) if cache < 1.0 else 1.0
        case = dict(path=path, graph=graph, batch=batch, fanouts=fanouts, cache=cache, gamma=gamma, padded=path != "fifo" and rng.random() < 0.6)
        if _fits(case):
            return case


# ---- inputs --------------------------------------------------------------------------------------------------------
_KEPT = {}                        # graphs and feature stores of this process


def _kept(key, make):
    if key not in _KEPT:
        _KEPT[key] = make()
    return _KEPT[key]


def _graph(name):
    w = get_config(name)
    return _kept(("graph", name), lambda: make_graph(w.num_nodes, w.mean_degree, w.d_min, w.d_max, w.a, w.symmetric, w.graph_seed,
                                                     w.idx_dtype, device="cuda"))


def _wide(case):
    w = get_config(case["graph"])
    elem = torch.empty(0, dtype=w.feat_dtype).element_size()
    return ((w.row_bytes + _LINE - 1) // _LINE * _LINE if case["padded"] else w.row_bytes) // elem


def _table(case):
    """[num_nodes, dim] rows on the GPU, row number = node id; N(0,1) values"""
    w = get_config(case["graph"])

    def make():
        gen = torch.Generator(device="cuda")
        gen.manual_seed(20)
        buf = torch.empty((w.num_nodes, _wide(case)), dtype=w.feat_dtype, device="cuda")
        step = 1 << 21
        for r in range(0, w.num_nodes, step):
            part = buf[r:r + step]
            part.copy_(torch.randn(part.shape, generator=gen, device="cuda"))
        return buf

    return _kept(("table", case["graph"], _wide(case)), make)[:, :w.feat_dim]


def _host_table(case):
    """the same rows in pinned host memory"""
    def make():
        full = _table(case)
        host = torch.empty((full.shape[0], full.stride(0)), dtype=full.dtype, pin_memory=True)
        host.copy_(full.as_strided(host.shape, full.stride()))
        return host
    return _kept(("host", case["graph"], _wide(case)), make)[:, :get_config(case["graph"]).feat_dim]


def _split(case):
    """(device map, device store): the rows of the nodes of highest degree in device memory in order of rank, the others in
    the host table at their id"""
    w = get_config(case["graph"])
    n_cached = min(w.num_nodes, math.ceil(case["cache"] * w.num_nodes))

    def make():
        order = torch.sort(_graph(case["graph"]).degrees(), descending=True, stable=True).indices
        cache_map = -torch.arange(w.num_nodes, dtype=torch.int32, device="cuda") - 1
        cache_map[order[:n_cached]] = torch.arange(n_cached, dtype=torch.int32, device="cuda")
        if n_cached == w.num_nodes:
            return cache_map, _table(case)   # row r of the table is as good as any other row
        full = _table(case)
        store = torch.zeros((n_cached, full.stride(0)), dtype=full.dtype, device="cuda")[:, :w.feat_dim]
        store.copy_(full[order[:n_cached]])
        return cache_map, store

    splits = [k for k in _KEPT if k[0] == "split" and k[1] != "citation"]
    key = ("split", case["graph"], n_cached, _wide(case))
    if key not in _KEPT and len(splits) > 6:
        del _KEPT[splits[0]]
    return _kept(key, make)


def _seed_nodes(case, base, number):
    w = get_config(case["graph"])
    return seed_batch(w.num_nodes, case["batch"], base, number, np.int32 if w.idx_dtype == torch.int32 else np.int64)


def _out_rows(case):
    """rows a caller sets aside: what the fanouts allow, never more than the graph has nodes"""
    return min(case["batch"] * math.prod(1 + f for f in _fanouts(case)), get_config(case["graph"]).num_nodes)


def _rows(case, n):
    w = get_config(case["graph"])
    return torch.zeros((n, _wide(case)), dtype=w.feat_dtype, device="cuda")[:, :w.feat_dim]


def _buffers(case):
    """the 32-bit and the 64-bit block arrays of the largest mini-batch that the fanouts allow, end to end"""
    w = get_config(case["graph"])
    dst, narrow, wide = case["batch"], 0, 0
    for f in _fanouts(case):
        narrow += dst + 1 + dst * f
        wide += dst * f
        dst = min(dst * (1 + f), w.num_nodes)
    more = (dst, 0) if w.idx_dtype == torch.int32 else (0, dst)
    return (torch.zeros(narrow + more[0], dtype=torch.int32, device="cuda"), torch.zeros(wide + more[1], dtype=torch.int64, device="cuda"))


def prepare(case, seed):
    w = get_config(case["graph"])
    fan = _fanouts(case)
    state = {"case": dict(case), "fanouts": fan, "rng": seed * 1000003 % (1 << 40), "bias": int(round(case["gamma"] * 65536)), "step": 0}
    if case["path"] == "ids":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        state["ids"] = torch.randint(0, w.num_nodes, (case["batch"],), generator=gen, device="cuda", dtype=w.idx_dtype)
        state["table"] = _table(case)
        state["ctx"] = a3.Context(1, [1])
        state["out"] = _rows(case, case["batch"])
        return state
    g = _graph(case["graph"])
    state["indptr"], state["indices"] = g.indptr, g.indices
    batches = {"fifo": _FIFO_BATCHES, "pipeline": _PIPE_BATCHES}.get(case["path"], 1)
    state["seeds"] = [torch.from_numpy(_seed_nodes(case, seed, b)).to("cuda") for b in range(batches)]
    state["buffers"] = [_buffers(case) for _ in range(_PIPE_BATCHES if case["path"] == "pipeline" else 1)]
    state["map"], state["dev"] = _split(case)
    state["host"] = _host_table(case) if case["cache"] < 1.0 or case["path"] == "fifo" else None
    if case["path"] == "pipeline":
        state["pipe"] = a3.Pipeline(a3.A3_PIPE_MODE1, _PIPE_WORKERS, case["batch"], fan)
        state["pipe"].reserve(w.num_nodes)
        rows = min(_out_rows(case), int(1.2 * _expected(case)[2]) + 4096)
        state["outs"] = [_rows(case, rows) for _ in range(_PIPE_BATCHES)]
        state["streams"] = [torch.cuda.ExternalStream(state["pipe"].stream(k)) for k in range(state["pipe"].n_workers)]
        torch.cuda.synchronize()
        return state
    # the map of a static fill does not change under the context; a FIFO cache's does
    state["ctx"] = a3.Context(case["batch"], fan, flags=a3.A3_STATIC_MAP if case["path"] in ("unit", "mean") and case["gamma"] > 1.0 else 0)
    state["ctx"].reserve(w.num_nodes)
    if case["path"] != "sample":
        state["out"] = _rows(case, _out_rows(case))
    if case["path"] == "mean":
        rows = min(case["batch"] * math.prod(1 + f for f in fan[:-1]), w.num_nodes)
        state["mean"] = _rows(case, rows)
    if case["path"] == "fifo":   # a ring as the static fill left it, oldest rows first
        n_slots = state["dev"].shape[0]
        state["map"], state["dev"] = state["map"].clone(), state["dev"].clone()
        state["owner"] = torch.empty(n_slots, dtype=torch.int32, device="cuda")
        nodes = torch.nonzero(state["map"] >= 0)[:, 0]
        state["owner"][state["map"][nodes].to(torch.int64)] = nodes.to(torch.int32)
        state["fifo"] = torch.zeros(4, dtype=torch.int32, device="cuda")
    return state


# ---- one pass ------------------------------------------------------------------------------------------------------
def _hand_over(b, buffers):
    """A mini-batch into the trainer's buffers, whose sizes do not change from one mini-batch to the next (ids, offsets and
    edge positions; the counts beside them say how much of the buffers is in use).  Rows have theirs already."""
    narrow = b.blk_indptr + b.blk_indices
    wide = list(b.blk_eids)
    (wide if b.input_nodes.dtype == torch.int64 else narrow).append(b.input_nodes)
    for parts, to in ((narrow, buffers[0]), (wide, buffers[1])):
        torch.cat(parts, out=to[:sum(len(p) for p in parts)])
    return {"narrow": buffers[0], "wide": buffers[1], "dst": b.n_dst, "edges": b.n_edges, "src": b.n_src}


def run(state):
    path = state["case"]["path"]
    if path == "ids":
        return state["ctx"].gather_features(state["table"], None, None, state["ids"], state["out"])
    if path == "pipeline":
        return _run_pipeline(state)
    ctx, seeds, rng = state["ctx"], state["seeds"][0], state["rng"]
    graph = (state["indptr"], state["indices"])
    if path == "sample":
        return _hand_over(ctx.sample_blocks(*graph, seeds, state["fanouts"], state["map"], state["bias"], rng), state["buffers"][0])
    more = {}
    if path == "split":
        ctx.sample_blocks_begin(*graph, seeds, state["fanouts"], state["map"], state["bias"], rng)
        ctx.gather_input_features(state["dev"], state["host"], state["map"], state["out"])
    else:
        if path == "fifo":
            k = state["step"]
            state["step"] = k + 1
            seeds, rng = state["seeds"][k % _FIFO_BATCHES], rng + k
        ctx.sample_gather_begin(*graph, seeds, state["fanouts"], state["map"], state["bias"], rng, state["dev"], state["host"], state["out"])
    if path == "mean":
        ctx.block_mean_of_hop(len(state["fanouts"]) - 1, state["out"], state["mean"])
        more = {"mean": state["mean"]}
    if path == "fifo":
        ctx.cache_fifo_update(state["map"], state["owner"], state["fifo"], state["dev"], state["out"], static_scratch=True)
        more = {"map": state["map"], "owner": state["owner"], "fifo": state["fifo"], "cache": state["dev"]}
    return {**_hand_over(ctx.sample_blocks_end(), state["buffers"][0]), "rows": state["out"], **more}


def _run_pipeline(state):
    pipe, got = state["pipe"], []

    def take():
        k = len(got)
        got.append({**_hand_over(pipe.wait(), state["buffers"][k]), "rows": state["outs"][k]})
        # the worker's next mini-batch overwrites the blocks: it starts behind the hand-over
        state["streams"][k % pipe.n_workers].wait_stream(torch.cuda.current_stream())

    for k in range(_PIPE_BATCHES):
        if k >= pipe.n_workers:
            take()
        pipe.submit(state["indptr"], state["indices"], state["seeds"][k], state["fanouts"], state["map"], state["bias"],
                    state["rng"] + k, state["dev"], None, state["outs"][k])
    while len(got) < _PIPE_BATCHES:
        take()
    return got
