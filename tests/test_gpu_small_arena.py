"""Preprocessing whose temporaries are carved from one block (up to 65536 pairs
and 32768 vertices) at the edges of that range, with odd sizes, and calls that
overlap on two streams. Against the oracle's CSR, ranks and T."""
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


def pairs(n, m):
    rng = np.random.default_rng(n + m)
    f = lambda: np.minimum((n * rng.random(m) ** 2).astype(np.int32), n - 1)
    return f(), f()


def same(tc, g, U):
    rp, col, perm = tc.tc_graph_export(g)
    assert np.array_equal(perm.cpu().numpy(), U.rank)
    assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
    assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
    assert int(tc.tc_count(g).item()) == oracle.count(U)


@pytest.mark.parametrize("n", [3, 701, 32767, 32768, 32769])
@pytest.mark.parametrize("m", [1, 16385, 16387, 40001, 65535, 65536, 65537])
def test_sizes(tc, n, m):
    print("case n=%d m=%d" % (n, m), flush=True)
    s, d = pairs(n, m)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    same(tc, g, oracle.preprocess(s, d, n))


def test_two_streams(tc):
    streams = [torch.cuda.Stream() for _ in range(2)]
    work = []
    for i in range(12):
        n, m = 900 + 613 * i, 16385 + 3001 * i
        s, d = pairs(n, m)
        ds, dd = torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda()
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[i % 2]):
            work.append((tc.tc_preprocess(ds, dd, n), oracle.preprocess(s, d, n), ds, dd))
    torch.cuda.synchronize()
    for g, U, _, _ in work:
        same(tc, g, U)
