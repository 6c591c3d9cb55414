"""What the server reserves for a graph that is being preprocessed is at least
what the call holds on the device: the uploaded pairs, the temporaries and the
graph. Small graphs (temporaries in one block) with few and with many pairs
per vertex, and the sizes just past them."""
import gc

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


def block_bytes(b):
    # the allocator's rounding: powers of two from 512 up to 1 MiB, then 2 MiB
    r = 512
    if b <= 1 << 20:
        while r < b:
            r *= 2
        return r
    return -(-b // (2 << 20)) * (2 << 20)


def graph(kind, n, m):
    rng = np.random.default_rng(n + m)
    if kind == "clique":  # as many vertices as m pairs join completely
        k = min(n, int((2 * m) ** 0.5))
        s, d = (x[:m].astype(np.int32) for x in np.triu_indices(k, 1))
        return s, d
    f = lambda: np.minimum((n * rng.random(m) ** (3 if kind == "skewed" else 1)).astype(np.int32), n - 1)
    return f(), f()


@pytest.mark.parametrize("kind", ["uniform", "skewed", "clique"])
@pytest.mark.parametrize("n", [64, 5000, 16384, 32768, 32769, 300000])
@pytest.mark.parametrize("m", [16, 1000, 16384, 16385, 40000, 65536, 65537, 200000])
def test_reserved_covers_the_build(tc, kind, n, m):
    s, d = graph(kind, n, m)
    m = len(s)
    ds, dd = torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda()
    torch.cuda.synchronize()
    gc.collect()
    tc.tc_release_cached_memory()
    base = tc.tc_memory_stats()
    assert base["cached"] == 0
    g = tc.tc_preprocess(ds, dd, n)
    st = tc.tc_memory_stats()
    held = st["in_use"] + st["cached"] - base["in_use"] + block_bytes(8 * m)
    g.free()
    with tc.Server(64 << 30, 4) as srv:
        srv.poll(srv.submit("count", s, d, n))
        reserved = srv.stats()["peak_reserved_bytes"]
    assert held <= reserved, (held, reserved)


@pytest.mark.parametrize("n,m", [(64, 65536), (4096, 32768), (32768, 1000), (32768, 65536), (300000, 1000000)])
def test_a_lone_graph_past_the_budget_is_built_lean(tc, n, m):
    # 56 bytes a pair, 40 a vertex and 1 MiB were enough to be admitted before
    # blocks and rounding counted, and still are for a request that is alone
    s, d = graph("uniform", n, m)
    budget = 56 * m + 40 * n + (1 << 20)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    want = int(tc.tc_count(g).item())
    with tc.Server(budget, 4) as srv:
        res = [srv.poll(t) for t in [srv.submit("count", s, d, n) for _ in range(3)]]
        st = srv.stats()
    assert [r["status"] for r in res] == [0, 0, 0] and [r["count"] for r in res] == [want] * 3
    with tc.Server(budget - 1, 4) as srv:
        r = srv.poll(srv.submit("count", s, d, n))
    assert r["status"] in (0, 2)


def test_cached_graphs_stay_when_a_request_cannot_fit(tc):
    s, d = graph("uniform", 4096, 32768)
    with tc.Server(64 << 20, 4) as srv:
        first = srv.poll(srv.submit("count", s, d, 4096, key=5))
        big = srv.poll(srv.submit("count", s, d, 1 << 28))  # 40 bytes a vertex: far past the budget
        again = srv.poll(srv.submit("count", None, None, 4096, key=5))
        st = srv.stats()
    assert first["status"] == 0 and big["status"] == 2
    assert again["status"] == 0 and again["count"] == first["count"]
    assert st["evicted"] == 0 and st["cache_hits"] == 1
