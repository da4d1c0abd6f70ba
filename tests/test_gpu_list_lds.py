"""Lists ranked in one workgroup's LDS at its edges: one list around 16384
nodes, batches whose longest list is around 4096 and 16384 nodes, more lists
than a workgroup takes at a time, empty lists, and malformed lists, which are
reported alone.  Ranks and statuses are exact."""

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


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 4096, 4097, 16383, 16384,
                               16385])
@pytest.mark.parametrize("to_tail", [False, True])
def test_one_list(pj, n, to_tail):
    succ = W.random_list(n, n)
    want = oracle.list_rank(succ)
    if to_tail:
        want = n - 1 - want
    st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    d = dev(np.concatenate([[0], succ]).astype(np.int32))[1:]   # not 16-byte aligned
    got = pj.list_rank(d, to_tail=to_tail, status=st)
    assert np.array_equal(got.cpu().numpy(), want) and int(st.item()) == pj.PJ_OK
    pj.list_rank(d, d, to_tail=to_tail)                          # in place
    assert np.array_equal(d.cpu().numpy(), want)


def lists_of(case):
    rng = np.random.default_rng(3)
    if case == "tiny":            # thousands of lists of 0..3 nodes
        sizes = rng.integers(0, 4, 5000)
    elif case == "mixed":
        sizes = (2.0 ** rng.uniform(0, 10, 700)).astype(int)
    else:
        sizes = np.array([5, 0, int(case), 1, 3000, int(case) - 1, 0, 77])
    return [W.random_list(int(s), 50 + i) for i, s in enumerate(sizes)]


@pytest.mark.parametrize("case", ["tiny", "mixed", "4096", "4097", "8192", "8193", "16384",
                                  "16385"])
@pytest.mark.parametrize("graph", [False, True])
def test_batches(pj, case, graph):
    lists = lists_of(case)
    succ, off = W.concat_lists([W.to_self_loop_tails(s) if i % 2 else s
                                for i, s in enumerate(lists)])
    want = np.concatenate([oracle.list_rank(s) for s in lists if len(s)])
    st = torch.full((len(lists),), 7, dtype=torch.int32, device="cuda")
    rank = torch.empty(int(off[-1]), dtype=torch.int32, device="cuda")
    d, o = dev(succ), dev(off)
    for _ in range(2):
        rank.fill_(-5)
        st.fill_(7)
        pj.list_rank_batched(d, o, rank, h_offsets=off, use_graph=graph, status=st)
        torch.cuda.synchronize()
        assert np.array_equal(rank.cpu().numpy(), want)
        assert (st.cpu().numpy() == pj.PJ_OK).all()
    pj.graph_cache_clear()


@pytest.mark.parametrize("case", ["cycle", "branch", "two_tails", "no_tail", "out_of_range",
                                  "range_as_tail", "negative"])
def test_malformed_list_is_reported_alone(pj, case):
    lists = lists_of("mixed")
    sizes = np.array([len(s) for s in lists])
    b = int(np.nonzero(sizes > 200)[0][1])
    n, s = int(sizes[b]), lists[b].copy()
    rank = oracle.list_rank(s)
    at = np.argsort(rank)                   # nodes from head to tail
    if case == "cycle":                     # the second half closes on itself
        s[at[n // 2 - 1]] = -1
        s[at[-1]] = at[n // 2]
    elif case == "branch":                  # two nodes with one successor, two heads
        s[at[3]] = at[9]
    elif case == "two_tails":
        s[at[5]] = -1
    elif case == "no_tail":
        s[at[-1]] = at[0]
    elif case == "out_of_range":
        s[at[5]] = n
    elif case == "range_as_tail":           # the tail itself points outside
        s[at[-1]] = n + 3
    else:
        s[at[5]] = -2
    lists[b] = s
    succ, off = W.concat_lists(lists)
    st = torch.full((len(lists),), 7, dtype=torch.int32, device="cuda")
    got = pj.list_rank_batched(dev(succ), dev(off), h_offsets=off, status=st).cpu().numpy()
    status = st.cpu().numpy()
    assert status[b] == pj.PJ_EBADLIST and (np.delete(status, b) == pj.PJ_OK).all()
    for i, l in enumerate(lists):
        if i != b and len(l):
            assert np.array_equal(got[off[i]:off[i + 1]], oracle.list_rank(l)), i
    # the list alone
    one = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    pj.list_rank(dev(s), status=one)
    assert int(one.item()) == pj.PJ_EBADLIST
    with pytest.raises(pj.PjError) as e:
        pj.list_rank(dev(s), validate=True)
    assert e.value.code == pj.PJ_EBADLIST
