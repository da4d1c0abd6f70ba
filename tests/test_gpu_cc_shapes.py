"""Components of graphs whose shape and ids make hooks meet: labels, and times
beside those of graphs of the same size that are easy."""

import time

import numpy as np
import pytest

import oracle

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


def solve_ms(pj, src, dst, n):
    """Time of a solve (the best of five); its labels are compared."""
    s, d = dev(src), dev(dst)
    label = torch.full((n,), -3, dtype=torch.int32, device="cuda")
    pj.connected_components(s, d, n, label)
    want = oracle.connected_components(np.ascontiguousarray(src, dtype=np.int32),
                                       np.ascontiguousarray(dst, dtype=np.int32), n)
    assert np.array_equal(label.cpu().numpy(), want)
    times = []
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        pj.connected_components(s, d, n, label)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    assert np.array_equal(label.cpu().numpy(), want)
    return 1e3 * min(times)


@pytest.mark.parametrize("n", [100_000, 1 << 20])
def test_hub(pj, n):
    i = np.arange(n - 1)
    first = solve_ms(pj, np.zeros(n - 1), i + 1, n)
    last = solve_ms(pj, np.full(n - 1, n - 1), i, n)   # every pair meets at the hub's parent
    assert last < 8 * max(first, 0.04), (first, last)
