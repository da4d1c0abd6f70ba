"""Performance cases: the calls a program makes of this library, over the
sizes and layouts of the benchmark and the tests.

Lists (int32 successor arrays) are ranked by the default method; components
take int32 pair arrays.  Sizes and layouts are the benchmark's (one list of
2^20 and 2^26 nodes, 4096 lists of 2^6..2^20 nodes, 1024 planted components of
2^22 vertices and 2^25 pairs in all, 1024 graphs of 2^8..2^16 vertices, 64 paths
with 8*10^6 pairs) and, below and between them, generic ones.
"""

import math
import random

import numpy as np
import torch

import paper_1002_4482_amd as pj

MAX_LIST = 1 << 26
MAX_BATCH_NODES = 1 << 28
MAX_PAIRS = 1 << 25


def listed():
    return [
        # one short list: a call inside a larger program, all latency
        {"name": "list_4096", "kind": "list", "n": 4096, "layout": "uniform", "to_tail": False},
        # an ordinary list of an odd size: a few dependent kernels
        {"name": "list_100003", "kind": "list", "n": 100_003, "layout": "uniform",
         "to_tail": False},
        # the benchmark's first list size
        {"name": "list_2p20", "kind": "list", "n": 1 << 20, "layout": "uniform",
         "to_tail": False},
        # the benchmark's headline list, four XCD-L2s past any cache but the last
        {"name": "list_2p26", "kind": "list", "n": 1 << 26, "layout": "uniform",
         "to_tail": False},
        # a list that was built mostly in memory order, ranked the paper's way
        # round (distance to the tail)
        {"name": "list_blocked_20000003", "kind": "list", "n": 20_000_003, "layout": "blocked",
         "to_tail": True},
        # prefix sums of node weights along a list
        {"name": "weighted_2p26", "kind": "weighted", "n": 1 << 26, "layout": "uniform"},
        # a forest of thousands of lists of every size in one call
        {"name": "batch_4096_lists", "kind": "batch", "count": 4096, "lo": 6.0, "hi": 20.0},
        # many short lists (chains of a hash table, polylines, queues)
        {"name": "batch_20000_short", "kind": "batch", "count": 20_000, "lo": 3.0, "hi": 10.0},
        # a small sparse graph: all latency
        {"name": "cc_1000", "kind": "cc", "graph": "uniform", "n": 1000, "m": 1500},
        # the benchmark's graph of 1024 components
        {"name": "cc_planted_2p22", "kind": "cc", "graph": "planted", "n": 1 << 22,
         "m": 1 << 25},
        # long paths, as sparse as a connected graph gets
        {"name": "cc_paths_8m", "kind": "cc", "graph": "paths", "n": 8_000_064,
         "m": 8_000_000},
        # a thousand graphs in one call
        {"name": "cc_batch_1024", "kind": "cc_batch", "count": 1024, "lo": 8.0, "hi": 16.0},
    ]


def draw(rng):
    kind = rng.choice(["list", "list", "weighted", "batch", "cc", "cc", "cc_batch"])

    def log_size(lo, hi):
        return max(1, int(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if kind == "list":
        return {"kind": kind, "n": log_size(1000, MAX_LIST),
                "layout": rng.choice(["uniform", "uniform", "uniform", "blocked", "sequential"]),
                "to_tail": rng.random() < 0.3}
    if kind == "weighted":
        return {"kind": kind, "n": log_size(1000, MAX_LIST),
                "layout": rng.choice(["uniform", "uniform", "blocked"])}
    if kind == "batch":
        hi = rng.uniform(6.0, 20.0)
        lo = rng.uniform(3.0, hi - 2.0)
        count = log_size(16, 20_000)
        return {"kind": kind, "count": min(count, max(1, int(MAX_BATCH_NODES / 2.0 ** hi))),
                "lo": lo, "hi": hi}
    if kind == "cc":
        graph = rng.choice(["uniform", "uniform", "planted", "paths", "trees"])
        if graph == "uniform":  # sparse enough that vertices stay alone
            n = log_size(1000, 1 << 22)
            return {"kind": kind, "graph": graph, "n": n, "m": int(n * rng.uniform(0.5, 2.5))}
        if graph == "planted":
            n = log_size(1000, 1 << 22)
            return {"kind": kind, "graph": graph, "n": n,
                    "m": min(MAX_PAIRS, int(n * rng.uniform(1.0, 8.0)))}
        n = log_size(1000, 8_000_064)
        return {"kind": kind, "graph": graph, "n": n, "m": n - min(64, n // 8)}
    hi = rng.uniform(8.0, 16.0)
    return {"kind": kind, "count": log_size(16, 1024), "lo": rng.uniform(4.0, hi - 1.0),
            "hi": hi}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _sizes(case, salt):
    """Instance sizes floor(2^U), U uniform: fixed by the case (the seed moves
    the contents)."""
    r = random.Random(f"{case['count']} {case['lo']} {case['hi']} {salt}")
    return np.array([int(2.0 ** r.uniform(case["lo"], case["hi"])) for _ in range(case["count"])],
                    dtype=np.int64)


def _offsets(sizes):
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    np.cumsum(sizes, out=off[1:])
    return off


def _order(case, seed):
    """The nodes of one list from head to tail."""
    n, layout = case["n"], case["layout"]
    if layout == "uniform":
        return torch.randperm(n, device="cuda", generator=_gen(seed))
    if layout == "sequential":  # in memory order from a random node round
        return (torch.arange(n, device="cuda") + random.Random(seed).randrange(n)) % n
    run = min(4096, max(1, n // 16))  # runs of consecutive ids, in random order
    runs = torch.randperm((n + run - 1) // run, device="cuda", generator=_gen(seed))
    order = (runs[:, None] * run + torch.arange(run, device="cuda")[None, :]).reshape(-1)
    return order[order < n]


def _succ(order):
    succ = torch.empty(order.numel(), dtype=torch.int32, device="cuda")
    succ[order[:-1]] = order[1:].to(torch.int32)
    succ[order[-1:]] = -1
    return succ


def _weights(case, seed):
    return torch.randint(0, 16, (case["n"],), dtype=torch.int32, device="cuda",
                         generator=_gen(seed + 7_000_001))


def _batch_order(off, seed):
    """Every list's nodes from head to tail, as global ids, list after list."""
    total = int(off[-1])
    sizes = torch.from_numpy(np.diff(off)).cuda()
    owner = torch.repeat_interleave(torch.arange(len(off) - 1, device="cuda"), sizes)
    key = torch.randint(0, 1 << 40, (total,), device="cuda", generator=_gen(seed))
    return torch.argsort(key.add_(owner << 40)), owner


def _batch_succ(off, seed):
    order, owner = _batch_order(off, seed)
    base = torch.from_numpy(off[:-1]).cuda()[owner]
    succ = torch.full((int(off[-1]),), -1, dtype=torch.int32, device="cuda")
    inside = owner[1:] == owner[:-1]  # consecutive places of one list
    succ[order[:-1][inside]] = (order[1:] - base[1:])[inside].to(torch.int32)
    return succ


def _rand_below(bound, g):
    """One uniform id in [0, bound) per entry of the tensor `bound`."""
    u = torch.rand(bound.numel(), dtype=torch.float64, device="cuda", generator=g)
    return torch.minimum((u * bound).to(torch.int64), bound - 1)


def _pairs(case, seed):
    n, m, g = case["n"], case["m"], _gen(seed)
    if case["graph"] == "uniform":
        return (torch.randint(0, n, (m,), dtype=torch.int32, device="cuda", generator=g),
                torch.randint(0, n, (m,), dtype=torch.int32, device="cuda", generator=g))
    label = torch.randperm(n, device="cuda", generator=g)
    pos = torch.arange(n, device="cuda")
    if case["graph"] == "paths":  # random paths: a permutation cut in n - m pieces
        cut = torch.randperm(n - 1, device="cuda", generator=g)[: n - m - 1]
        keep = torch.ones(n - 1, dtype=torch.bool, device="cuda")
        keep[cut] = False
        a, b = pos[:-1][keep], pos[1:][keep]
    elif case["graph"] == "trees":  # n - m complete binary trees
        per = (n + (n - m) - 1) // (n - m)
        at = pos % per
        a = pos[at > 0]
        b = a - at[at > 0] + (at[at > 0] - 1) // 2
        a, b = a[:m], b[:m]
    else:  # planted: groups of log-uniform size, a random tree and more pairs in each
        r = random.Random(f"{n} {m}")
        groups = max(1, min(1024, n // 16))
        raw = np.array([2.0 ** (16.0 * r.random()) for _ in range(groups)])
        sizes = np.maximum(1, np.floor(raw / raw.sum() * (n - groups))).astype(np.int64)
        sizes[int(np.argmax(sizes))] += n - int(sizes.sum())
        size = torch.from_numpy(sizes).cuda()
        start = torch.cumsum(size, 0) - size
        group = torch.repeat_interleave(torch.arange(groups, device="cuda"), size)
        within = pos - start[group]
        a = pos[within > 0]
        b = a - within[a] + _rand_below(within[a], g)
        u = torch.randint(0, n, (m - a.numel(),), device="cuda", generator=g)
        v = start[group[u]] + _rand_below(size[group[u]], g)
        a, b = torch.cat([a, u]), torch.cat([b, v])
    shuffle = torch.randperm(a.numel(), device="cuda", generator=g)
    return label[a[shuffle]].to(torch.int32), label[b[shuffle]].to(torch.int32)


def _graph_offsets(case):
    """Offset tables of a batch of graphs: sizes and average degrees 2..16."""
    sizes = _sizes(case, "graphs")
    r = random.Random(f"{case['count']} {case['lo']} {case['hi']} degree")
    pairs = np.array([int(round(s * r.uniform(2.0, 16.0) / 2)) for s in sizes], dtype=np.int64)
    return _offsets(sizes), _offsets(pairs)


def _batch_pairs(voff, eoff, seed):
    bound = torch.repeat_interleave(torch.from_numpy(np.diff(voff)).cuda(),
                                    torch.from_numpy(np.diff(eoff)).cuda())
    g = _gen(seed)
    return _rand_below(bound, g).to(torch.int32), _rand_below(bound, g).to(torch.int32)


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind}
    if kind in ("list", "weighted"):
        state["succ"] = _succ(_order(case, seed))
        state["to_tail"] = case.get("to_tail", False)
        if kind == "weighted":
            state["weight"] = _weights(case, seed)
    elif kind == "batch":
        off = _offsets(_sizes(case, "lists"))
        state.update(succ=_batch_succ(off, seed), h_off=off, off=torch.from_numpy(off).cuda())
    elif kind == "cc":
        state["src"], state["dst"] = _pairs(case, seed)
        state["n"] = case["n"]
    else:
        voff, eoff = _graph_offsets(case)
        state["src"], state["dst"] = _batch_pairs(voff, eoff, seed)
        state.update(h_voff=voff, h_eoff=eoff, voff=torch.from_numpy(voff).cuda(),
                     eoff=torch.from_numpy(eoff).cuda())
    return state


def run(state):
    kind = state["kind"]
    if kind == "list":
        return pj.list_rank(state["succ"], to_tail=state["to_tail"])
    if kind == "weighted":
        return pj.list_rank_weighted(state["succ"], state["weight"])
    if kind == "batch":
        return pj.list_rank_batched(state["succ"], state["off"], h_offsets=state["h_off"])
    if kind == "cc":
        return pj.connected_components(state["src"], state["dst"], state["n"])
    return pj.connected_components_batched(state["src"], state["dst"], state["voff"],
                                           state["eoff"], h_vtx_off=state["h_voff"],
                                           h_edge_off=state["h_eoff"])


def work(case):
    """Every input word read once, every output word written once; integer
    work only."""
    kind = case["kind"]
    if kind == "list":
        moved = 8 * case["n"]
    elif kind == "weighted":
        moved = 12 * case["n"]
    elif kind == "batch":
        moved = 8 * int(_sizes(case, "lists").sum()) + 8 * (case["count"] + 1)
    elif kind == "cc":
        moved = 8 * case["m"] + 4 * case["n"]
    else:
        voff, eoff = _graph_offsets(case)
        moved = 8 * int(eoff[-1]) + 4 * int(voff[-1]) + 16 * (case["count"] + 1)
    return {"bytes": moved, "flops": 0}


# ------------------------------------------------------------- exact results
def _min_labels(u, v, n):
    """Smallest vertex id of each vertex's component: hook every root to the
    smallest neighbouring root, jump pointers, repeat."""
    label = torch.arange(n, device="cuda")
    while u.numel():
        lu, lv = label[u], label[v]
        differ = lu != lv
        u, v, lu, lv = u[differ], v[differ], lu[differ], lv[differ]
        label.scatter_reduce_(0, torch.maximum(lu, lv), torch.minimum(lu, lv), "amin")
        while True:
            jumped = label[label]
            if torch.equal(jumped, label):
                break
            label = jumped
    return label


def exact(case, seed):
    kind = case["kind"]
    if kind in ("list", "weighted"):
        order = _order(case, seed)
        rank = torch.empty(case["n"], dtype=torch.int64, device="cuda")
        if kind == "weighted":
            w = _weights(case, seed).to(torch.int64)[order]
            rank[order] = torch.cumsum(w, 0) - w
        else:
            place = torch.arange(case["n"], device="cuda")
            rank[order] = case["n"] - 1 - place if case["to_tail"] else place
        return rank
    if kind == "batch":
        off = _offsets(_sizes(case, "lists"))
        order, owner = _batch_order(off, seed)
        rank = torch.empty(int(off[-1]), dtype=torch.int64, device="cuda")
        base = torch.from_numpy(off[:-1]).cuda()[owner]
        rank[order] = torch.arange(int(off[-1]), device="cuda") - base
        return rank
    if kind == "cc":
        src, dst = _pairs(case, seed)
        return _min_labels(src.to(torch.int64), dst.to(torch.int64), case["n"])
    voff, eoff = _graph_offsets(case)
    src, dst = _batch_pairs(voff, eoff, seed)
    pair_base = torch.repeat_interleave(torch.from_numpy(voff[:-1]).cuda(),
                                        torch.from_numpy(np.diff(eoff)).cuda())
    base = torch.repeat_interleave(torch.from_numpy(voff[:-1]).cuda(),
                                   torch.from_numpy(np.diff(voff)).cuda())
    return _min_labels(pair_base + src, pair_base + dst, int(voff[-1])) - base
