"""Components at the edges of the solver's paths: chunks of 2048 pairs, parts
of the pairs (2 m < 3 n or not), class bytes (n >= 3 * 2^19, m >= 3 n) used and
not used, and chains as long as the graph.  Labels are exact."""

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
