"""Per-vertex counts at the edges of the range whose counters are kept in copies
(8192 highest ranks), against the oracle, integer by integer."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


def graph(n, m, seed):
    rng = np.random.default_rng(seed)
    f = lambda: np.minimum((n * rng.random(m) ** 3).astype(np.int32), n - 1)
    return f(), f()


def build(tc, s, d, n):
    return oracle.preprocess(s, d, n), tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)


@pytest.mark.parametrize("n", [2, 100, 8191, 8192, 8193, 8300, 40000])
def test_vertex_counts(tc, n):
    print("case n=%d" % n, flush=True)
    s, d = graph(n, 14 * n, n + 1)
    U, g = build(tc, s, d, n)
    full = oracle.support(U, oracle.MODE_FULL)[1][:U.m].astype(np.int64)
    rows = np.repeat(np.arange(n), np.diff(U.row_ptr))
    by_rank = (np.bincount(rows, full, n) + np.bincount(U.col[:U.m], full, n)).astype(np.int64) // 2
    tri = tc.tc_vertex_triangles(g).cpu().numpy()
    assert np.array_equal(tri, by_rank[U.rank])
    assert tc.tc_transitivity(g) >= 0
