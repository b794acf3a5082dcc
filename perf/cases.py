"""The workloads by which the speed of this library is judged.

Each case is one pass of work that a program with a dynamic graph on the GPU has the library do,
through the entry points of `paper_2504_10233_amd` and with the library's default tuning: walk
queries (DeepWalk, node2vec, personalized PageRank), batched and streaming updates, and the build.
Graphs, weight laws and batches are those of `bench.py` and the tests (R-MAT and Erdos-Renyi graphs
of 16 edges per vertex, uniform, Zipf and lognormal weights, planted hubs), from the generators in
`synth/`, on the GPU.

Updates slide a window over the graph's own edge list: its `parts` parts are all in the graph but
one, a pass inserts the missing part and deletes the next one.  So the graph keeps its size however
often a pass is repeated, inserts follow the graph's degree law, deletes name existing edges, and
every pass is a batch that the graph has not seen in its present state.  A pass ends with short walks
from updated vertices, which see every edge, weight and group the batch has changed there.

Every output is whole numbers (vertex ids, visit counts, statistics) that the random stream of
(seed, walk id, step) fixes bit for bit.
"""
import math

import torch

import synth
from paper_2504_10233_amd import Graph, ppr_threshold, quantize_biases

DEV = "cuda:0"
EDGES_PER_VERTEX = 16
PROBE_WALKS = 1 << 17  # walks that read back what an update batch changed


def listed():
    return [
        # The smallest query: the tests' plain-method graph, one launch and its latency.
        {"name": "walk_small", "kind": "walk", "n": 1000, "m": 10000, "graph": "er", "weights": "uniform16",
         "bias": "int", "walks": 1000, "length": 80},
        # Embedding of a whole graph: one walk of 80 steps from each vertex (bench.py --workload deepwalk).
        {"name": "walk_all", "kind": "walk", "n": 1 << 22, "m": 1 << 26, "graph": "rmat", "weights": "zipf",
         "bias": "int", "walks": 1 << 22, "length": 80},
        # The same with floating-point biases (fixed point, 8 fraction bits), a sample of the vertices.
        {"name": "walk_float", "kind": "walk", "n": 1 << 18, "m": 1 << 22, "graph": "rmat", "weights": "zipf",
         "bias": "float", "walks": 50001, "length": 80},
        # Second-order walks at the usual p and q.
        {"name": "node2vec", "kind": "node2vec", "n": 1 << 20, "m": 1 << 24, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "walks": 100000, "length": 80, "p": 0.5, "q": 2.0},
        # An interactive recommendation: personalized PageRank of a few vertices.
        {"name": "ppr_few", "kind": "ppr", "n": 1 << 18, "m": 1 << 22, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "sources": 10, "per_source": 1000, "stop": 0.15},
        # The headline query of bench.py: 10^4 sources, 10^7 walks on R-MAT 24.
        {"name": "ppr_many", "kind": "ppr", "n": 1 << 24, "m": 1 << 28, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "sources": 10000, "per_source": 1000, "stop": 0.15},
        # The dynamic loop of bench.py: a query whose histograms are left running beside the next batch.
        {"name": "step", "kind": "step", "n": 1 << 21, "m": 1 << 25, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "sources": 1000, "per_source": 1000, "stop": 0.15, "records": 100000, "parts": 4},
        # A trickle of changes, as a serving loop applies them between queries.
        {"name": "update_small", "kind": "update", "n": 1 << 18, "m": 1 << 22, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "records": 100, "parts": 8},
        # The headline batch of bench.py: 10^6 records on R-MAT 24.
        {"name": "update_large", "kind": "update", "n": 1 << 24, "m": 1 << 28, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "records": 1000000, "parts": 4},
        # Updates that fall on hubs (bench.py --workload skewed-updates): four of five records on
        # planted hubs of up to 3 x 10^5 edges, heavy-tailed weights.
        {"name": "update_hubs", "kind": "update", "n": 1 << 20, "m": 1 << 24, "graph": "hubs", "weights": "lognormal",
         "bias": "int", "records": 10000, "parts": 4},
        # Changes that have to be applied one by one, in their order.
        {"name": "stream", "kind": "stream", "n": 1 << 20, "m": 1 << 24, "graph": "rmat", "weights": "uniform24",
         "bias": "int", "records": 20000, "parts": 4},
        # A graph that is loaded, walked once and dropped.
        {"name": "build", "kind": "build", "n": 1 << 20, "m": 1 << 24, "graph": "rmat", "weights": "zipf",
         "bias": "int"},
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["walk", "walk", "node2vec", "ppr", "ppr", "step", "update", "update", "update", "stream",
                       "build"])
    top = {"walk": 22, "node2vec": 20, "ppr": 23, "step": 21, "update": 22, "stream": 20, "build": 20}[kind]
    n = _log(rng, 1 << 10, 1 << top)
    case = {"kind": kind, "n": n, "m": int(n * rng.uniform(6, EDGES_PER_VERTEX)), "graph": rng.choice(["rmat", "rmat", "er"]),
            "weights": rng.choice(["uniform16", "uniform24", "zipf", "lognormal"]), "bias": "int"}
    if kind == "walk":
        case["bias"] = rng.choice(["int", "int", "float", "alias"])
        case.update(walks=_log(rng, 100, n), length=rng.randint(5, 80))
    elif kind == "node2vec":
        case.update(walks=_log(rng, 100, 100000), length=rng.randint(5, 80), p=rng.choice([0.5, 1.0, 4.0]),
                    q=rng.choice([0.5, 2.0]))
    elif kind == "ppr":
        case["sources"] = _log(rng, 1, min(10000, n // 4))
        case.update(per_source=_log(rng, 50, 1000), stop=rng.choice([0.15, 0.15, 1 / 40]))
    elif kind == "step":
        case["sources"] = _log(rng, 10, min(1000, n // 4))
        case.update(per_source=_log(rng, 50, 1000), stop=0.15, parts=4)
    elif kind == "update":
        case["bias"] = rng.choice(["int", "int", "int", "float", "alias"])
        if rng.random() < 0.3 and n <= 1 << 20:
            case["graph"] = "hubs"
        case["parts"] = rng.choice([4, 8])
    elif kind == "stream":
        case["parts"] = 4
    if kind in ("step", "update", "stream"):
        most = {"step": 100000, "update": 1000000, "stream": 20000}[kind]
        case["records"] = _log(rng, 2, min(most, case["m"] // 4))
    return case


# ---------------------------------------------------------------------------------------------- inputs
def _edges(case, seed):
    """(src, dst, hubs) on the GPU; hubs: the ids of planted hubs, or None."""
    n, m = case["n"], case["m"]
    if case["graph"] == "er":
        return (*synth.er_graph(n, m, seed, device=DEV), None)
    src, dst = synth.rmat_graph(max(1, (n - 1).bit_length()), m, seed, device=DEV)
    src, dst = src % n, dst % n
    if case["graph"] != "hubs":
        return src, dst, None
    # as in bench.py, one hub per 10^4 vertices, of 3 x 10^4 to 3 x 10^5 edges where the graph has a
    # million vertices, fewer edges in a smaller one
    top = math.log10(0.3 * n)
    hubs, hs, hd = synth.planted_hubs(n, max(4, n // 10000), top - 1, top, seed, device=DEV)
    return torch.cat([src, hs]), torch.cat([dst, hd]), hubs


def _weights(case, m, seed):
    law = case["weights"]
    if law == "zipf":
        w = synth.weights_zipf(m, 1.5, (1 << 20) - 1, seed, device=DEV)
    elif law == "lognormal":
        w = synth.weights_lognormal(m, 8.0, 3.0, seed, device=DEV, hi=2**24 - 1 if case["bias"] == "float" else 2**32 - 1)
    else:
        w = synth.weights_uniform(m, 1, 1 << (16 if law == "uniform16" else 24), seed, device=DEV)
    if case["bias"] == "float":
        bias = (w.to(torch.float64).clamp_(max=2**23) + synth.uniform_f64(seed, 77, m, device=DEV)).to(torch.float32)
        return quantize_biases(bias, 1.0, 8)
    return _i32(w)


def _i32(x):
    """int64 values as int32 bit patterns, the form in which the library takes them without a copy."""
    return torch.where(x >= 2**31, x - 2**32, x).to(torch.int32).contiguous()


def _graph(case, src, dst, w):
    return Graph(case["n"], src, dst, w, device=DEV, frac_bits=8 if case["bias"] == "float" else 0,
                 alias_table=case["bias"] == "alias")


def _window(case, src, dst, w, hubs, seed):
    """The window's parts: [(insert src, dst, weights), ...] and the edges that start in the graph."""
    half, parts = max(1, case["records"] // 2), case["parts"]
    if hubs is None:
        pick = synth.EdgeMirror._distinct(torch.arange(src.numel(), device=DEV), half * parts, seed, 30)
    else:
        on = torch.isin(src, hubs)
        most = int(0.8 * half) * parts
        a = synth.EdgeMirror._distinct(torch.nonzero(on).flatten(), most, seed, 30)
        b = synth.EdgeMirror._distinct(torch.nonzero(~on).flatten(), half * parts - a.numel(), seed, 31)
        pick = torch.cat([a, b])
        pick = pick[torch.argsort(synth.uniform_u32(seed, 32, pick.numel(), DEV))]
    half = pick.numel() // parts
    cut = [pick[i * half:(i + 1) * half] for i in range(parts)]
    keep = torch.ones(src.numel(), dtype=torch.bool, device=DEV)
    keep[cut[0]] = False
    return [(src[c].contiguous(), dst[c].contiguous(), w[c].contiguous()) for c in cut], keep


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    seed = seed * 8
    src, dst, hubs = _edges(case, seed)
    w = _weights(case, src.numel(), seed + 1)
    src, dst = _i32(src), _i32(dst)
    state = {"case": case, "seed": seed + 2, "pass": 0}
    if kind == "build":
        state.update(src=src, dst=dst, w=w, starts=torch.arange(n, dtype=torch.int32, device=DEV))
        return state
    if kind in ("update", "stream", "step"):
        state["window"], keep = _window(case, src, dst, w, hubs, seed + 3)
        state["graph"] = _graph(case, src[keep], dst[keep], w[keep])
        if kind == "stream":
            # inserts and deletes mixed, one order per part
            half = state["window"][0][0].numel()
            state["order"] = torch.argsort(synth.uniform_u32(seed + 4, 1, 2 * half, DEV))
            state["op"] = (state["order"] >= half).to(torch.int32)
    else:
        state["graph"] = _graph(case, src, dst, w)
    if kind in ("ppr", "step"):
        live = torch.nonzero(torch.bincount(src.long(), minlength=n) > 0).flatten()
        order = torch.argsort(synth.uniform_u32(seed + 5, 1, live.numel(), DEV))
        state["sources"] = live[order[: case["sources"]]].to(torch.int32).contiguous()
        state["stop"] = ppr_threshold(case["stop"])
        state["beside"] = torch.cuda.Stream() if kind == "step" else None
        # the program's own result buffers, with room for every visit being to another vertex
        walks = case["sources"] * case["per_source"]
        state["found"] = torch.zeros((2, int(1.25 * walks / case["stop"]) + 4096), dtype=torch.int32, device=DEV)
    if kind in ("walk", "node2vec"):
        walks = case["walks"]
        starts = torch.arange(n, device=DEV) if walks == n else synth.below(seed + 6, 1, walks, n, DEV)
        state["starts"] = starts.to(torch.int32).contiguous()
    return state


# ------------------------------------------------------------------------------------------------ a pass
def _batch(state):
    """The next records of the window: the part to insert and the part to delete."""
    parts = state["window"]
    i = state["pass"] % len(parts)
    return parts[i], parts[(i + 1) % len(parts)]


def _changes(stats):
    """What an update call reports (how many entries it read to find its deletes is no result)."""
    return [stats["inserted"], stats["deleted"], stats["not_found"], stats["touched_vertices"], stats["transitions"]]


def _seen(state, ins, dele):
    """Short walks from updated vertices."""
    starts = torch.cat([ins[0][: PROBE_WALKS // 2], dele[0][: PROBE_WALKS // 2]])
    return state["graph"].walk(starts, 4, state["seed"])


def _collect(state, off, vtx, cnt):
    """The histograms in the program's buffers (what lies behind off[-1] there is of no meaning)."""
    found = state["found"]
    k = min(vtx.numel(), found.shape[1])
    found[0, :k].copy_(vtx[:k])
    found[1, :k].copy_(cnt[:k])
    return off, found


def run(state):
    case, seed, g = state["case"], state["seed"], state.get("graph")
    kind = case["kind"]
    if kind == "walk":
        return g.walk(state["starts"], case["length"], seed)
    if kind == "node2vec":
        return g.node2vec(state["starts"], case["length"], seed, case["p"], case["q"])
    if kind == "ppr":
        off, vtx, cnt, steps = g.ppr(state["sources"], case["per_source"], state["stop"], 200, seed)
        return steps, _collect(state, off, vtx, cnt)
    if kind == "build":
        g = _graph(case, state["src"], state["dst"], state["w"])
        out = g.walk(state["starts"], 4, seed)
        g.close()
        return out
    ins, dele = _batch(state)
    state["pass"] += 1
    if kind == "update":
        stats = g.update(*ins, dele[0], dele[1])
        return _changes(stats), _seen(state, ins, dele)
    if kind == "stream":
        src, dst, w = (torch.cat([a, b])[state["order"]] for a, b in zip(ins, dele))
        stats = g.update_stream(state["op"], src, dst, w)
        return _changes(stats), _seen(state, ins, dele)
    # step: the query's histograms run beside the batch
    steps = g.ppr_async(state["sources"], case["per_source"], state["stop"], 200, seed, hist_stream=state["beside"])
    stats = g.update(*ins, dele[0], dele[1])
    return steps, _changes(stats), _collect(state, *g.ppr_result())


# ------------------------------------------------------------------------------------------------ work
def work(case):
    """Bytes of one pass.  A transition reads one 64-byte line of its vertex's sampling space and one
    edge word, but no vertex and no edge needs to be read more than once; an update record reads and
    writes one such line and one edge word with its sequence number."""
    n, m, kind = case["n"], case["m"], case["kind"]
    bias = {"int": 0, "float": 0, "alias": 16}[case["bias"]]

    def transitions(t):
        return min(t * (64.0 + 8 + bias), n * (64.0 + 16 * bias) + 8.0 * m)

    total = 0.0
    if kind in ("walk", "node2vec"):
        total = transitions(case["walks"] * case["length"]) + 4.0 * case["walks"] * (case["length"] + 2)
    if kind in ("ppr", "step"):
        walks = case["sources"] * case["per_source"]
        visits = walks / case["stop"]
        total = transitions(visits) + 4.0 * case["sources"] + 8.0 * visits
    if kind in ("update", "stream", "step"):
        half = max(1, case["records"] // 2)
        total += half * (12 + 8 + 2 * 2 * (64.0 + 12))
        if kind != "step":
            total += transitions(min(PROBE_WALKS, 2 * half) * 4) + min(PROBE_WALKS, 2 * half) * 24.0
    if kind == "build":
        total = 12.0 * m + 64.0 * n + 12.0 * m + 24.0 * n
    return {"bytes": total, "flops": 0.0}


def exact(case, seed):
    """None: no output is a rounded number (see the top of this file)."""
    return None
