"""Components at the edges of the solver's paths: chunks of 2048 pairs, parts
of the pairs (2 m < 3 n or not), class bytes (n >= 3 * 2^19, m >= 3 n) used and
not used, chains as long as the graph, and the one-workgroup solver (16384 and
65536 vertices, rows and chunks of pairs, 512 graphs at a time, heavy graphs
first).  Labels are exact."""

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
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def solve(pj, src, dst, n):
    out = pj.connected_components(dev(src), dev(dst), n)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def device_wide_graph(case):
    if case.startswith("chunk"):        # around one chunk, more vertices than LDS holds
        n, m = 70_000, int(case[5:])
        return (*W.random_graph(n, m, m), n)
    if case == "dense_chunk":           # parts of one chunk: no chunk for the swaps
        n, m = 66_000, 99_000
        return (*W.random_graph(n, m, 3), n)
    if case == "classes_used":
        n = (3 << 19) + 1
        src, dst, _ = W.planted_graph(n, 3 * n + 5, 7, 11)
        return src, dst, n
    if case == "classes_not_used":      # components of at most 64 vertices
        n, c = 3 << 19, 64
        rng = np.random.default_rng(12)
        src = rng.integers(0, n, 3 * n + 2047)
        dst = src // c * c + rng.integers(0, c, src.shape[0])
        return src, dst, n
    i = np.arange(300_000)
    if case == "path_doubled":          # blind hooks chain every vertex to the one before
        return np.tile(i, 2), np.tile(i + 1, 2), 300_001
    if case == "path_shuffled":
        p = np.random.default_rng(13).permutation(4 * i.shape[0])
        return np.tile(i, 4)[p], np.tile(i + 1, 4)[p], 300_001
    w = 550                             # grid
    g = np.arange(w * w).reshape(w, w)
    return (np.concatenate([g[:, :-1].ravel(), g[:-1].ravel()]),
            np.concatenate([g[:, 1:].ravel(), g[1:].ravel()]), w * w)


@pytest.mark.parametrize("case", ["chunk1", "chunk2047", "chunk2048", "chunk2049", "dense_chunk",
                                  "classes_used", "classes_not_used", "path_doubled",
                                  "path_shuffled", "grid"])
def test_device_wide_path(pj, case):
    src, dst, n = device_wide_graph(case)
    want = oracle.connected_components(src.astype(np.int32), dst.astype(np.int32), n)
    assert np.array_equal(solve(pj, src, dst, n), want)


@pytest.mark.parametrize("n,m", [(1, 1), (2, 3), (63, 64), (500, 511), (500, 512), (500, 513),
                                 (16384, 20_000), (16385, 20_000), (65_535, 30_001),
                                 (65_536, 70_000), (65_537, 30_000)])
def test_one_workgroup_graph(pj, n, m):
    src, dst = W.random_graph(n, m, n + 7 * m)
    src[-1] = dst[-1] = n - 1           # the last vertex is read and written
    assert np.array_equal(solve(pj, src, dst, n), oracle.connected_components(src, dst, n))


def test_one_workgroup_chain(pj):
    n = 65_536                          # blind hooks make one chain of the whole LDS
    i = np.arange(n - 1, dtype=np.int32)
    assert (solve(pj, i, i + 1, n) == 0).all()
    back = i[::-1].copy()
    assert (solve(pj, back + 1, back, n) == 0).all()


def batch(case):
    rng = np.random.default_rng(5)
    if case == "tiny":                  # more graphs than one workgroup takes at a time
        sizes = rng.integers(0, 4, 1500)
        pairs = np.where(sizes > 0, rng.integers(0, 5, 1500), 0)
    elif case == "capacity":            # a graph that fills LDS between small ones
        sizes = np.array([100, 0, 65_536, 1, 65_535, 2000, 16_384])
        pairs = np.array([150, 0, 70_000, 2, 66_000, 0, 20_001])
    elif case == "heavy":               # more workgroups than CUs and a few heavy graphs
        sizes = np.concatenate([rng.integers(100, 4000, 400), [30_000, 50, 40_000]])
        pairs = np.concatenate([rng.integers(100, 4000, 400), [50_000, 60, 80_000]])
    else:                               # one graph too large for LDS: all device-wide
        sizes = np.array([300, 65_537, 40])
        pairs = np.array([400, 80_000, 50])
    voff = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    eoff = np.concatenate([[0], np.cumsum(pairs)]).astype(np.int64)
    bound = np.repeat(sizes, pairs)
    src = (rng.random(bound.shape[0]) * bound).astype(np.int32)
    dst = (rng.random(bound.shape[0]) * bound).astype(np.int32)
    return src, dst, voff, eoff


@pytest.mark.parametrize("case", ["tiny", "capacity", "heavy", "too_large"])
@pytest.mark.parametrize("tables", ["host", "device", "graph"])
def test_batch_of_one_workgroup_graphs(pj, case, tables):
    src, dst, voff, eoff = batch(case)
    G = voff.shape[0] - 1
    want = oracle.connected_components_batched(src, dst, voff, eoff)
    bad = int(np.argmax(np.diff(eoff)))           # and then one pair out of range
    broken = dst.copy()
    broken[eoff[bad]] = voff[bad + 1] - voff[bad]
    kw = {} if tables == "device" else {"h_vtx_off": voff, "h_edge_off": eoff}
    if tables == "graph":
        kw["use_graph"] = True
    st = torch.empty(G, dtype=torch.int32, device="cuda")
    ds, dd = dev(src), dev(dst)
    dv, de = torch.from_numpy(voff).cuda(), torch.from_numpy(eoff).cuda()
    lab = torch.empty(int(voff[-1]), dtype=torch.int32, device="cuda")
    for pairs, code in ((dst, pj.PJ_OK), (broken, pj.PJ_EINVAL), (dst, pj.PJ_OK)):
        dd.copy_(dev(pairs))
        lab.fill_(-1)
        st.fill_(7)
        pj.connected_components_batched(ds, dd, dv, de, lab, status=st, **kw)
        torch.cuda.synchronize()
        got, status = lab.cpu().numpy(), st.cpu().numpy()
        assert status[bad] == code and (np.delete(status, bad) == pj.PJ_OK).all()
        keep = np.ones(got.shape[0], dtype=bool)
        if code != pj.PJ_OK:
            keep[voff[bad]:voff[bad + 1]] = False
        assert np.array_equal(got[keep], want[keep])
    pj.graph_cache_clear()


# deep trees for the shortcut: chains in id order, up and down, beside pairs that
# hook blind, at sizes around a workgroup's 1024 vertices
@pytest.mark.parametrize("n", [65_537, 66_560, 66_561, 100_000, (1 << 20) + 1023, 1 << 22])
@pytest.mark.parametrize("shape", ["up", "down", "doubled", "x4", "comb"])
def test_deep_trees(pj, n, shape):
    a = np.arange(n - 1, dtype=np.int32)
    src, dst = a, a + 1
    if shape == "down":
        src, dst = dst[::-1], src[::-1]
    elif shape == "doubled":
        src, dst = np.concatenate([src, dst]), np.concatenate([dst, src])
    elif shape == "x4":
        perm = np.random.default_rng(n).permutation(n - 1)
        src, dst = np.tile(src[perm], 4), np.tile(dst[perm], 4)
    elif shape == "comb":               # a chain of the even ids, a tooth at each
        a = np.arange(0, n - 2, 2, dtype=np.int32)
        t = np.arange(0, n - 1, 2, dtype=np.int32)
        src, dst = np.concatenate([a, t]), np.concatenate([a + 2, t + 1])
    want = oracle.connected_components(src, dst, n)
    assert np.array_equal(solve(pj, src, dst, n), want)


def test_one_workgroup_chain_and_more_pairs(pj):
    n = 65_536                          # one chain of the whole LDS, and pairs beside it
    i = np.arange(n - 1, dtype=np.int32)
    far = np.random.default_rng(4).integers(0, n, (2, 6000)).astype(np.int32)
    for a, b in ((i, i + 1), (i[::-1] + 1, i[::-1])):
        src, dst = np.concatenate([a, far[0]]), np.concatenate([b, far[1]])
        assert (solve(pj, src, dst, n) == 0).all()


# both sides of the choice between one workgroup and the device
@pytest.mark.parametrize("n,m", [(27_000, 27_000), (29_000, 28_900), (40_000, 39_000),
                                 (40_000, 41_000), (60_000, 76_000), (60_000, 89_990),
                                 (60_000, 90_000), (30_000, 80_000), (30_000, 99_000)])
def test_either_path(pj, n, m):
    src, dst = W.random_graph(n, m, n + m)
    assert np.array_equal(solve(pj, src, dst, n), oracle.connected_components(src, dst, n))
