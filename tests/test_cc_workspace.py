"""Workspace of the components calls: the reported bytes are what the solve
takes, enough for either entry point, and less is refused whichever path a graph
would take."""

import numpy as np
import pytest

import oracle
import workloads as W
from paper_1002_4482_amd import _lib

torch = pytest.importorskip("torch")


def reported(n, m, G=1):
    return _lib.load().pj_cc_workspace_bytes(n, m, G, None)


@pytest.mark.parametrize("n,m,G", [(0, 0, 1), (1, 0, 1), (1000, 1500, 1), (1 << 22, 1 << 25, 1),
                                   (8_000_064, 8_000_000, 1), (11_000_000, 47_000_000, 1024),
                                   (1 << 30, 1 << 34, 1)])
def test_reported_bytes(n, m, G):
    # a batch's pairs rewritten, a byte per vertex, a word per 2048 pairs and per graph
    got = reported(n, m, G)
    assert 8 * m <= got <= 8 * m + n + m // 512 + 4 * G + 8192


@pytest.fixture(scope="module")
def pj():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1002_4482_amd as pj
    pj.load()
    return pj


# one workgroup's LDS, and device-wide without and with class bytes
@pytest.mark.gpu
@pytest.mark.parametrize("n,m", [(1000, 1500), (70_000, 90_000), (3 << 19, 9 << 19)])
@pytest.mark.parametrize("batched", [False, True])
def test_sizes(pj, n, m, batched):
    src, dst = W.random_graph(n, m, 3)
    want = oracle.connected_components(src, dst, n)
    s, d = torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda()
    voff, eoff = np.array([0, n], np.int64), np.array([0, m], np.int64)
    tables = [torch.from_numpy(t).cuda() for t in (voff, eoff)]

    def call(nbytes):
        # a guard behind the workspace
        mem = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        if batched:
            got = pj.connected_components_batched(s, d, *tables, h_vtx_off=voff, h_edge_off=eoff,
                                                  workspace=mem[:nbytes])
        else:
            got = pj.connected_components(s, d, n, workspace=mem[:nbytes])
        assert bool((mem[nbytes:] == 0x5A).all())
        return got.cpu().numpy()

    assert np.array_equal(call(reported(n, m)), want)
    with pytest.raises(pj.PjError) as e:
        call(256)
    assert e.value.code == pj.PJ_EINVAL


@pytest.mark.gpu
def test_a_budget_admits_what_fits(pj):
    from paper_1002_4482_amd import serve
    n, m = 1 << 16, 1 << 18
    src, dst = W.random_graph(n, m, 5)
    # pairs, their rewritten copy, labels and tables: 4.6 MiB
    with serve.Server(hbm_budget=5 << 20, max_inflight=2, max_batch=4) as srv:
        st, _, out = srv.wait(srv.submit_cc(src, dst, n), timeout_s=60)
        assert st == 0 and np.array_equal(out, oracle.connected_components(src, dst, n))
        assert srv.stats()["bytes_peak"] <= 5 << 20
