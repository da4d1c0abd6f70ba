"""Batches with many empty and tiny instances in one place, beside long ones:
results and statuses, and that they cost no more than a few times what the same
instances spread over the batch do."""

import time

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pj():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1002_4482_amd as pj
    pj.load()
    return pj


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def best_ms(f):
    f()
    times = []
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return 1e3 * min(times)


def lists_in_place(longs, size, empties, where):
    """`longs` lists of `size` nodes, the empty ones in one place or spread."""
    if where == "together":
        sizes = np.concatenate([np.full(longs // 2, size), np.zeros(empties, np.int64),
                                np.full(longs - longs // 2, size)])
    else:
        sizes = np.zeros(longs + empties, np.int64)
        sizes[np.linspace(0, longs + empties - 1, longs).astype(int)] = size
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    one = [W.random_list(size, s) for s in range(8)]
    want = [oracle.list_rank(s) for s in one]
    succ = np.concatenate([one[i % 8] for i in range(longs)])
    return succ, off, np.concatenate([want[i % 8] for i in range(longs)])


# the recorded walk (2^16 nodes a list end on its chunks' borders), and lists in
# LDS with its two workgroup sizes
@pytest.mark.parametrize("longs,size,empties", [(256, 1 << 16, 1_000_000), (300, 1000, 1_000_000),
                                                (60, 9000, 1_000_000)])
def test_lists(pj, longs, size, empties):
    ms = {}
    for where in ("together", "spread"):
        succ, off, want = lists_in_place(longs, size, empties, where)
        d, o = dev(succ), dev(off)
        rank = torch.full_like(d, -3)
        st = torch.full((len(off) - 1,), 7, dtype=torch.int32, device="cuda")
        ms[where] = best_ms(lambda: pj.list_rank_batched(d, o, rank, h_offsets=off, status=st))
        assert np.array_equal(rank.cpu().numpy(), want)
        assert (st.cpu().numpy() == pj.PJ_OK).all()
    assert ms["together"] < 4 * ms["spread"], ms


# graphs of few vertices and many pairs, of one vertex, and empty ones in one
# place: chunks of pairs that hold hundreds of graphs, and thousands that hold one
@pytest.mark.parametrize("case", ["dense", "one_vertex", "empty", "pairs_behind"])
@pytest.mark.parametrize("how", ["host", "device", "graph"])
def test_graphs(pj, case, how):
    rng = np.random.default_rng(3)
    if case == "dense":
        sizes, pairs = np.full(20, 100), np.full(20, 200_000)
    elif case == "one_vertex":
        sizes, pairs = np.ones(100_000, np.int64), rng.integers(0, 3, 100_000)
    elif case == "empty":
        sizes = np.concatenate([np.full(60, 900), np.zeros(300_000, np.int64), np.full(60, 3000)])
        pairs = sizes * 3 // 2
    else:                       # all the pairs in the last of many graphs
        sizes, pairs = np.full(3000, 50), np.zeros(3000, np.int64)
        pairs[-5:] = 300_000
    voff = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    eoff = np.concatenate([[0], np.cumsum(pairs)]).astype(np.int64)
    bound = np.repeat(sizes, pairs)
    src = (rng.random(bound.shape[0]) * bound).astype(np.int32)
    dst = (rng.random(bound.shape[0]) * bound).astype(np.int32)
    want = oracle.connected_components_batched(src, dst, voff, eoff)
    kw = {} if how == "device" else {"h_vtx_off": voff, "h_edge_off": eoff}
    if how == "graph":
        kw["use_graph"] = True
    st = torch.full((len(sizes),), 7, dtype=torch.int32, device="cuda")
    label = torch.full((int(voff[-1]),), -3, dtype=torch.int32, device="cuda")
    args = [dev(a) for a in (src, dst, voff, eoff)]
    for _ in range(2):
        pj.connected_components_batched(*args, label, status=st, **kw)
        torch.cuda.synchronize()
        assert np.array_equal(label.cpu().numpy(), want)
        assert (st.cpu().numpy() == pj.PJ_OK).all()
    pj.graph_cache_clear()
