"""Workspaces kept between calls: more streams than blocks, threads that share a
stream, and blocks given back between calls.  Every result is compared."""

import threading

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


@pytest.fixture(scope="module")
def lists():
    out = []
    for i, n in enumerate([16_385, 17_003, 20_000, 33_000, 48_001, 70_000]):
        succ = W.random_list(n, 90 + i)
        out.append((torch.from_numpy(succ).cuda(), torch.from_numpy(oracle.list_rank(succ)).cuda()))
    torch.cuda.synchronize()
    return out


def test_more_streams_than_blocks(pj, lists):
    streams = [torch.cuda.Stream() for _ in range(20)]
    ranks = []
    for k in range(100):
        d, want = lists[k % len(lists)]
        out = torch.full_like(d, -7)
        out.record_stream(streams[k % 20])
        streams[k % 20].wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(streams[k % 20]):
            pj.list_rank(d, out)
        ranks.append((out, want))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in ranks)


@pytest.mark.parametrize("shared", [True, False])
def test_threads(pj, lists, shared):
    one = torch.cuda.Stream()
    bad = []

    def work(t):
        stream = one if shared else torch.cuda.Stream()
        with torch.cuda.stream(stream):
            got = []
            for k in range(40):
                d, want = lists[(t + k) % len(lists)]
                got.append((pj.list_rank(d), want))
            stream.synchronize()
            if not all(torch.equal(a, b) for a, b in got):
                bad.append(t)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not bad


def test_given_back(pj, lists):
    for _ in range(3):
        for d, want in lists:
            assert torch.equal(pj.list_rank(d), want)
        pj.graph_cache_clear()
