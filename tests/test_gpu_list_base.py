"""The base of the recursion (a level of at most 16384 nodes ranked in one
workgroup's LDS) for one list and for few and many lists, at levels of a few
to 16384 nodes, weighted, and on splitter lists that are no lists."""

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


# spacing 2 and a cutoff of 16384 make the base about half the list
@pytest.mark.parametrize("n", [16385, 20_003, 24_576, 32_000, 32_766])
@pytest.mark.parametrize("layout", ["random", "sequential"])
def test_one_list(pj, n, layout):
    succ = W.random_list(n, n) if layout == "random" else W.sequential_list(n)
    st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    got = pj.list_rank(dev(succ), spacing=2, status=st)
    assert np.array_equal(got.cpu().numpy(), oracle.list_rank(succ))
    assert int(st.item()) == pj.PJ_OK
    # a base of a few nodes
    got = pj.list_rank(dev(succ), spacing=4096, cutoff=64, status=st)
    assert np.array_equal(got.cpu().numpy(), oracle.list_rank(succ))
    w = np.random.default_rng(n).integers(0, 50_000, n).astype(np.int32)
    got = pj.list_rank_weighted(dev(succ), dev(w), spacing=2, status=st)
    assert np.array_equal(got.cpu().numpy(), oracle.list_rank_weighted(succ, w))
    assert int(st.item()) == pj.PJ_OK


# both kernels: up to 1024 lists and more
@pytest.mark.parametrize("L", [2, 1023, 1024, 1025, 3000])
def test_batches(pj, L):
    rng = np.random.default_rng(L)
    sizes = rng.integers(0, 12, L)
    sizes[L // 2] = 17_000              # too long for one workgroup's lists
    succ, off = W.concat_lists([W.random_list(int(s), 9 + i) for i, s in enumerate(sizes)])
    st = torch.full((L,), 7, dtype=torch.int32, device="cuda")
    got = pj.list_rank_batched(dev(succ), dev(off), h_offsets=off, status=st)
    assert oracle.list_rank_batched(succ, off)[0].max() == 0
    assert np.array_equal(got.cpu().numpy(), oracle.list_rank_batched(succ, off)[1])
    assert (st.cpu().numpy() == pj.PJ_OK).all()


@pytest.mark.parametrize("case", ["cycle", "branch", "two_tails"])
def test_malformed(pj, case):
    n = 20_000
    succ = W.random_list(n, 5)
    at = np.argsort(oracle.list_rank(succ))
    if case == "cycle":
        succ[at[n // 2 - 1]] = -1
        succ[at[-1]] = at[n // 2]
    elif case == "branch":
        succ[at[100]] = at[9000]
    else:
        succ[at[5000]] = -1
    st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    for spacing in (2, 8):
        pj.list_rank(dev(succ), spacing=spacing, status=st)
        assert int(st.item()) == pj.PJ_EBADLIST


# 10240 nodes: one splitter per 4 ids up to there, per 8 beyond
@pytest.mark.parametrize("n", [20_475, 20_476, 20_477, 20_478, 20_479, 20_480, 20_481, 20_483])
def test_block_edges(pj, n):
    succ = W.random_list(n, n)
    st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    got = pj.list_rank(dev(succ), spacing=2, status=st)
    assert np.array_equal(got.cpu().numpy(), oracle.list_rank(succ))
    assert int(st.item()) == pj.PJ_OK
    succ[np.argsort(oracle.list_rank(succ))[n // 3]] = -1
    pj.list_rank(dev(succ), spacing=2, status=st)
    assert int(st.item()) == pj.PJ_EBADLIST
