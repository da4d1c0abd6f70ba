"""One list of at most 16384 nodes, weighted or of more than 4096, ranked by one
kernel: sizes around its rows and splitter blocks, both rank origins, in place,
unaligned arrays, and every way of not being one list."""

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 5, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 5000, 10239, 10240, 10241,
         10243, 16383, 16384]


@pytest.fixture(scope="module")
def pj():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1002_4482_amd as pj
    pj.load()
    return pj


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def status():
    return torch.full((1,), 7, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("layout", ["random", "sequential", "reversed", "self_tail"])
def test_ranks(pj, n, layout):
    if layout == "sequential":
        succ = W.sequential_list(n)
    elif layout == "reversed":
        succ = np.arange(n, dtype=np.int32) - 1
    else:
        succ = W.random_list(n, n)
        if layout == "self_tail":
            at = int(np.flatnonzero(succ == -1)[0])
            succ[at] = at
    want = oracle.list_rank(succ)
    st = status()
    assert np.array_equal(pj.list_rank(dev(succ), status=st).cpu().numpy(), want)
    assert int(st.item()) == pj.PJ_OK
    assert np.array_equal(pj.list_rank(dev(succ), to_tail=True).cpu().numpy(), n - 1 - want)
    w = np.random.default_rng(n).integers(-1000, 100_000, n).astype(np.int32)
    st = status()
    got = pj.list_rank_weighted(dev(succ), dev(w), status=st).cpu().numpy()
    assert np.array_equal(got, oracle.list_rank_weighted(succ, w))
    assert int(st.item()) == pj.PJ_OK
    # in place, one word into the arrays
    d = dev(np.concatenate([[0], succ]).astype(np.int32))
    pj.list_rank(d[1:], d[1:])
    assert np.array_equal(d[1:].cpu().numpy(), want)
    d = dev(np.concatenate([[0], succ]).astype(np.int32))
    pj.list_rank_weighted(d[1:], dev(np.concatenate([[0], w]).astype(np.int32))[1:], d[1:])
    assert np.array_equal(d[1:].cpu().numpy(), oracle.list_rank_weighted(succ, w))


@pytest.mark.parametrize("n", [2, 3, 64, 4097, 10240, 16384])
@pytest.mark.parametrize("case", ["cycle", "whole_cycle", "branch", "to_head", "two_tails",
                                  "past_end", "below"])
def test_not_one_list(pj, n, case):
    succ = W.random_list(n, n + 1)
    at = np.argsort(oracle.list_rank(succ))
    if case == "cycle":             # the second half closes on itself
        succ[at[n // 2 - 1]] = -1
        succ[at[-1]] = at[n // 2]
        if n == 2:
            succ[:] = [1, 0]
        elif n // 2 == n - 1:       # (a cycle of one node is a tail)
            succ[at[n // 2 - 1]] = at[-1]
            succ[at[-1]] = at[0]
    elif case == "whole_cycle":
        succ[at[-1]] = at[0]
    elif case == "branch":
        succ[at[0]] = at[-1]
        if n == 2:
            succ[:] = [-1, -1]
    elif case == "to_head":
        succ[at[n // 2]] = at[0]
        if n // 2 == 0:
            succ[:] = [1, 0]
    elif case == "two_tails":
        succ[at[0]] = -1
    elif case == "past_end":
        succ[at[0]] = n
    else:
        succ[at[0]] = -2
    try:
        oracle.list_rank(succ)
        pytest.skip("still one list")
    except Exception:
        pass
    w = np.ones(n, dtype=np.int32)
    for run in (lambda st: pj.list_rank(dev(succ), status=st),
                lambda st: pj.list_rank_weighted(dev(succ), dev(w), status=st)):
        st = status()
        run(st)
        assert int(st.item()) == pj.PJ_EBADLIST
