"""Small graphs whose degree counters take more LDS from call to call (4 bytes a
vertex, 64 to 128 KiB), smallest first: every launch may take what it needs,
whatever size the process saw first. Against the oracle."""
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


def test_growing_vertex_counts(tc):
    for n in (16383, 16385, 20000, 27001, 32767, 32768):
        print("case n=%d" % n, flush=True)
        rng = np.random.default_rng(n)
        s, d = (rng.integers(0, n, 5 * n).astype(np.int32) for _ in range(2))
        s[0], d[0] = n - 1, n - 2  # the last counters are used
        U = oracle.preprocess(s, d, n)
        g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
        rp, col, perm = tc.tc_graph_export(g)
        assert np.array_equal(perm.cpu().numpy(), U.rank)
        assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
        assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
