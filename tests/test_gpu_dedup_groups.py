"""Duplicates of graphs past 32768 vertices are found in LDS, in groups of keys
that agree in the sort's top bits: sizes at the edges of a tile (4096 keys),
groups that run on past it, a group past the limit (one edge more than 2^20
times: the keys are then sorted by all bits), one vertex that all edges start
at, self loops, both directions of every edge; ids that take every count of
sort passes. Against the oracle: CSR, ranks and T."""
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


def check(tc, s, d, n):
    s, d = np.ascontiguousarray(s, dtype=np.int32), np.ascontiguousarray(d, dtype=np.int32)
    U = oracle.preprocess(s, d, n)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    rp, col, perm = tc.tc_graph_export(g)
    assert np.array_equal(perm.cpu().numpy(), U.rank)
    assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
    assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
    assert int(tc.tc_count(g).item()) == oracle.count(U)


def pairs(n, m, seed):
    rng = np.random.default_rng(seed)
    f = lambda: np.minimum((n * rng.random(m) ** 2).astype(np.int64), n - 1)
    return f(), f()


@pytest.mark.parametrize("m", [1, 2, 4095, 4096, 4097, 4159, 4160, 4161, 8192, 100001])
def test_pair_counts(tc, m):
    print("case m=%d" % m, flush=True)
    check(tc, *pairs(40000, m, m), 40000)


@pytest.mark.parametrize("n,m", [(32769, 70000), (65536, 70000), (65537, 70000), (1 << 20, 300000), ((1 << 24) + 1, 70000),
                                 (20, 1 << 21), (200, 1200000), (1000, 1200000), (3000, 2500000)])
def test_vertex_counts(tc, n, m):
    print("case n=%d m=%d" % (n, m), flush=True)
    check(tc, *pairs(n, m, n), n)


@pytest.mark.parametrize("copies", [64, 4000, 5000, (1 << 20) - 5000, (1 << 20) + 9000])
def test_one_edge_many_times(tc, copies):
    print("case copies=%d" % copies, flush=True)
    s, d = pairs(50000, 60000, 1)
    at = np.random.default_rng(2).integers(0, s.size, copies)
    check(tc, np.insert(s, at, 7), np.insert(d, at, 4321), 50000)


@pytest.mark.parametrize("case", ["star_low", "star_high", "both_ways", "loops", "one_loop", "path"])
def test_shapes(tc, case):
    print("case %s" % case, flush=True)
    n = 70000
    s, d = pairs(n, 90000, 3)
    leaf = np.arange(n)
    if case == "star_low":
        s, d = np.concatenate([np.zeros(n - 1, np.int64), s]), np.concatenate([leaf[1:], d])
    elif case == "star_high":
        s, d = np.concatenate([np.full(n - 1, n - 1), s]), np.concatenate([leaf[:-1], d])
    elif case == "both_ways":
        s, d = np.concatenate([s, d, s]), np.concatenate([d, s, d])
    elif case == "loops":
        s, d = np.concatenate([s, leaf, leaf]), np.concatenate([d, leaf, leaf])
    elif case == "one_loop":
        s, d = np.concatenate([s, np.full(1200000, n - 1)]), np.concatenate([d, np.full(1200000, n - 1)])
    else:
        s, d = np.concatenate([leaf[:-1], leaf[:-2]]), np.concatenate([leaf[1:], leaf[2:]])
    check(tc, s, d, n)
