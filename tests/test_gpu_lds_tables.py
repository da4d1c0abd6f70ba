"""Device offset tables that are not the ones the host planned with, on the LDS
paths of lists and graphs: entries that decrease, jump past LDS or past the
arrays.  Every instance gets a status, those at a wrong entry an error, and
nothing outside the arrays is written."""

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GUARD = 1 << 16
BIG = np.iinfo(np.int64)


@pytest.fixture(scope="module")
def pj():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1002_4482_amd as pj
    pj.load()
    return pj


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def spoilt(off, case):
    """The table with some entries changed, and the instances beside them."""
    off = off.copy()
    G = len(off) - 1
    at = [3, G // 2, G // 2 + 7, G - 3]
    if case == "jump":          # far ahead and back again: {0, 5, 100000, 10}
        off[at] = off[-1] - 7
    elif case == "back":
        off[at] = 1
    elif case == "negative":
        off[at] = -5
    elif case == "outside":
        off[at] = off[-1] + 9
    elif case == "extremes":
        off[at] = [BIG.max - 2, BIG.min + 2, BIG.max, BIG.min]
    else:
        off[1:-1] = off[1:-1][::-1].copy()
        at = range(1, G)
    return off, sorted({g for i in at for g in (i - 1, i)})


def guarded(n):
    t = torch.full((n + 2 * GUARD,), -9, dtype=torch.int32, device="cuda")
    return t, t[GUARD:GUARD + n]


def untouched(t, n):
    return bool((t[:GUARD] == -9).all()) and bool((t[GUARD + n:] == -9).all())


CASES = ["jump", "back", "negative", "outside", "extremes", "reversed"]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("longest", [3000, 9000])
@pytest.mark.parametrize("graph", [False, True])
def test_lists(pj, case, longest, graph):
    sizes = np.random.default_rng(1).integers(1, 200, 3000)
    sizes[[50, 1500, 2900]] = longest
    succ, off = W.concat_lists([W.random_list(int(s), i) for i, s in enumerate(sizes)])
    n, L = int(off[-1]), len(sizes)
    table, beside = spoilt(off, case)
    whole, rank = guarded(n)
    st_whole, st = guarded(L)
    d, o = dev(succ), dev(off)
    status, want = oracle.list_rank_batched(succ, off)
    for spoil in (False, True, False):
        o.copy_(dev(table if spoil else off))
        rank.fill_(-3)
        st.fill_(7)
        pj.list_rank_batched(d, o, rank, h_offsets=off, status=st, use_graph=graph)
        torch.cuda.synchronize()
        got = st.cpu().numpy()
        assert untouched(whole, n) and untouched(st_whole, L)
        if not spoil:
            assert (got == pj.PJ_OK).all() and np.array_equal(rank.cpu().numpy(), want)
        else:
            assert np.isin(got, [pj.PJ_OK, pj.PJ_EBADLIST]).all()
            if case != "reversed":
                assert (got == pj.PJ_EBADLIST)[beside].all()
    pj.graph_cache_clear()


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("which", ["vertices", "pairs", "both"])
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("heavy", [False, True])
def test_graphs(pj, case, which, graph, heavy):
    rng = np.random.default_rng(2)
    sizes = rng.integers(1, 400, 3000)
    pairs = rng.integers(0, 600, 3000)
    if heavy:                   # more workgroups than CUs, and heavy graphs among them
        sizes[[50, 1500, 2900]] = 20_000
        pairs[[50, 700, 1500, 2900]] = 30_000
    voff = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    eoff = np.concatenate([[0], np.cumsum(pairs)]).astype(np.int64)
    bound = np.repeat(sizes, pairs)
    src = (rng.random(bound.shape[0]) * bound).astype(np.int32)
    dst = (rng.random(bound.shape[0]) * bound).astype(np.int32)
    want = oracle.connected_components_batched(src, dst, voff, eoff)
    n, G = int(voff[-1]), len(sizes)
    vt = spoilt(voff, case)[0] if which != "pairs" else voff
    et = spoilt(eoff, case)[0] if which != "vertices" else eoff
    whole, label = guarded(n)
    st_whole, st = guarded(G)
    s, d, dv, de = dev(src), dev(dst), dev(voff), dev(eoff)
    for spoil in (False, True, False):
        dv.copy_(dev(vt if spoil else voff))
        de.copy_(dev(et if spoil else eoff))
        label.fill_(-3)
        st.fill_(7)
        pj.connected_components_batched(s, d, dv, de, label, h_vtx_off=voff, h_edge_off=eoff,
                                        status=st, use_graph=graph)
        torch.cuda.synchronize()
        got = st.cpu().numpy()
        assert untouched(whole, n) and untouched(st_whole, G)
        if not spoil:
            assert (got == pj.PJ_OK).all() and np.array_equal(label.cpu().numpy(), want)
        else:
            assert np.isin(got, [pj.PJ_OK, pj.PJ_EINVAL]).all()
            if case in ("negative", "outside", "extremes"):
                assert (got == pj.PJ_EINVAL).any()
    pj.graph_cache_clear()
