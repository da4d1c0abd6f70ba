"""The recorded level-0 walk (nodes recorded in strips, dealt to bins of 32768
ids and put in order in LDS) at its edges: the sizes where it starts, batches
whose lists fill, straddle and miss bins, cut walks, both rank origins, in
place, a caller workspace too small for it, graph replay, and malformed lists."""

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


@pytest.mark.parametrize("n", [(11 << 20) - 1, 11 << 20, (11 << 20) + 32769])
@pytest.mark.parametrize("to_tail", [False, True])
def test_one_list(pj, n, to_tail):
    succ, order = W.random_list_with_order(n, n)
    want = np.empty(n, dtype=np.int32)
    want[order] = np.arange(n)[::-1] if to_tail else np.arange(n)
    st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    d = dev(succ)
    got = pj.list_rank(d, to_tail=to_tail, status=st)
    assert np.array_equal(got.cpu().numpy(), want) and int(st.item()) == pj.PJ_OK
    # many cuts, and walks of any length
    for kw in (dict(max_walk=16), dict(spacing=4096), dict(spacing=2), dict(max_walk=100)):
        got = pj.list_rank(d, to_tail=to_tail, status=st, **kw)
        assert np.array_equal(got.cpu().numpy(), want) and int(st.item()) == pj.PJ_OK, kw
    pj.list_rank(d, d, to_tail=to_tail, status=st)      # in place
    assert np.array_equal(d.cpu().numpy(), want) and int(st.item()) == pj.PJ_OK


def test_local_list_takes_the_other_path(pj):
    n = 12_000_000
    succ, order = W.blocked_list_with_order(n, 4096, 3)
    want = np.empty(n, dtype=np.int32)
    want[order] = np.arange(n)
    d = dev(succ)
    assert np.array_equal(pj.list_rank(d).cpu().numpy(), want)
    pj.list_rank(d, d)
    assert np.array_equal(d.cpu().numpy(), want)


def sizes_of(case):
    rng = np.random.default_rng(8)
    if case == "bins":           # whole bins, one more and one less, empty lists
        return np.array([32768] * 8 + [32769, 0, 32767, 1, 0, 65536, 20_000] * 6 + [100_000] * 4)
    if case == "mixed":          # many short lists beside long ones
        return np.concatenate([rng.integers(0, 40, 3000), [1 << 20, 300_000],
                               rng.integers(0, 3000, 500), [17_000]])
    if case == "start":          # 2^20 nodes in all
        return np.array([500_000, (1 << 20) - 500_000])
    return np.array([1 << 21, 5, (1 << 21) - 1])  # the longest lists it takes


@pytest.mark.parametrize("case", ["bins", "mixed", "start", "long"])
@pytest.mark.parametrize("how", ["plain", "to_tail", "in_place", "graph", "workspace", "cuts"])
def test_batches(pj, case, how):
    sizes = sizes_of(case)
    succ, off = W.concat_lists([W.random_list(int(s), 70 + i) for i, s in enumerate(sizes)])
    L = len(sizes)
    status, want = oracle.list_rank_batched(succ, off)
    assert (status == 0).all()
    if how == "to_tail":
        want = np.repeat(sizes, sizes).astype(np.int32) - 1 - want
    d, o = dev(succ), dev(off)
    st = torch.full((L,), 7, dtype=torch.int32, device="cuda")
    kw = dict(h_offsets=off, status=st)
    if how == "to_tail":
        kw["to_tail"] = True
    if how == "graph":
        kw["use_graph"] = True
    if how == "cuts":
        kw["max_walk"] = 32
    if how == "workspace":       # as much as the walk in place needs
        from paper_1002_4482_amd import _lib
        kw["workspace"] = torch.empty(
            _lib.load().pj_list_rank_workspace_bytes(int(off[-1]), L, None), dtype=torch.uint8,
            device="cuda")
    rank = d if how == "in_place" else torch.empty_like(d)
    for _ in range(1 if how == "in_place" else 3):
        st.fill_(7)
        pj.list_rank_batched(d, o, rank, **kw)
        torch.cuda.synchronize()
        assert np.array_equal(rank.cpu().numpy(), want)
        assert (st.cpu().numpy() == pj.PJ_OK).all()
        if how != "in_place":
            rank.fill_(-3)
    pj.graph_cache_clear()


@pytest.mark.parametrize("case", ["cycle", "branch", "two_tails", "out_of_range", "all_to_one"])
@pytest.mark.parametrize("batched", [False, True])
def test_malformed(pj, case, batched):
    n = (1 << 20) + 5 if batched else (11 << 20) + 7
    succ, order = W.random_list_with_order(n, 4)
    if case == "cycle":
        succ[order[n // 2 - 1]] = -1
        succ[order[-1]] = order[n // 2]
    elif case == "branch":
        succ[order[100]] = order[9000]
    elif case == "two_tails":
        succ[order[5000]] = -1
    elif case == "out_of_range":
        succ[order[5000]] = n
    else:
        succ[:] = 77
        succ[77] = -1
    if batched:
        other = W.random_list(40_000, 6)
        s, off = W.concat_lists([other, succ, other])
        st = torch.full((3,), 7, dtype=torch.int32, device="cuda")
        pj.list_rank_batched(dev(s), dev(off), h_offsets=off, status=st)
        assert int(st[1].item()) == pj.PJ_EBADLIST
    else:
        st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
        pj.list_rank(dev(succ), status=st)
        assert int(st.item()) == pj.PJ_EBADLIST


# entries of one word and of two: bins of 2^15 nodes up to lists of 2^17, then
# smaller ones, pairs beyond 2^20
@pytest.mark.parametrize("longest", [1 << 12, 1 << 17, (1 << 17) + 1, (1 << 19) + 5, 1 << 20,
                                     (1 << 20) + 1, 1 << 21])
@pytest.mark.parametrize("to_tail", [False, True])
def test_entry_widths(pj, longest, to_tail):
    sizes = [1, longest, 0, longest - 1, 4095, longest, 2] + [3000] * 400
    succ, off = W.concat_lists([W.random_list(s, 31 + i) for i, s in enumerate(sizes)])
    st = torch.full((len(sizes),), 7, dtype=torch.int32, device="cuda")
    got = pj.list_rank_batched(dev(succ), dev(off), h_offsets=off, to_tail=to_tail, status=st)
    bad, want = oracle.list_rank_batched(succ, off)
    if to_tail:
        want = np.repeat(np.diff(off), np.diff(off)) - 1 - want
    assert bad.max() == 0
    assert np.array_equal(got.cpu().numpy(), want)
    assert (st.cpu().numpy() == pj.PJ_OK).all()
