"""Lists without a tail on the LDS path, long enough for distances round a
cycle to pass 16 bits: the tail linked back into the list, or to its head.  The
status says so without the full check, and lists beside them are not touched."""

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


def broken(n, shape, seed):
    if shape == "descending":       # a cycle of 2^k neighbours and a way into it
        s = np.arange(n, dtype=np.int32) - 1
        s[0] = (1 << (n - 1).bit_length() - 1) - 1
        return s
    s, order = W.random_list_with_order(n, seed)
    s[order[-1]] = order[0 if shape == "circle" else np.random.default_rng(seed).integers(n - 1)]
    return s


@pytest.mark.parametrize("shape", ["back", "circle", "descending"])
@pytest.mark.parametrize("n", [1000, 4095, 4096, 5000, 16384])
def test_one_list(pj, n, shape):
    st = torch.empty(1, dtype=torch.int32, device="cuda")
    for seed in range(1 if shape == "descending" else 40):
        d = dev(broken(n, shape, seed))
        for _ in range(3):          # waves meet in another order each time
            st.fill_(7)
            pj.list_rank(d, status=st)
            assert int(st.item()) == pj.PJ_EBADLIST, seed


@pytest.mark.parametrize("shape", ["back", "circle", "descending"])
@pytest.mark.parametrize("n", [1000, 4000, 4096, 8000, 16384])
@pytest.mark.parametrize("graph", [False, True])
def test_beside_valid_lists(pj, n, shape, graph):
    lists = [W.random_list(s, s) for s in (300, n, 5, 2000, n)]
    seeds = range(40)
    lists += [broken(n, shape, s) for s in seeds]
    order = np.random.default_rng(n).permutation(len(lists))
    bad = order >= len(lists) - len(seeds)
    lists = [lists[i] for i in order]
    succ, off = W.concat_lists(lists)
    st = torch.empty(len(lists), dtype=torch.int32, device="cuda")
    d, o = dev(succ), dev(off)
    rank = torch.empty_like(d)
    for _ in range(3):
        st.fill_(7)
        pj.list_rank_batched(d, o, rank, h_offsets=off, status=st, use_graph=graph)
        torch.cuda.synchronize()
        assert np.array_equal(st.cpu().numpy(), np.where(bad, pj.PJ_EBADLIST, pj.PJ_OK))
        got = rank.cpu().numpy()
        for i in np.flatnonzero(~bad):
            assert np.array_equal(got[off[i]:off[i + 1]], oracle.list_rank(lists[i])), i
    pj.graph_cache_clear()
