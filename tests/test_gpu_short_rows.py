"""Short rows: the rows of U whose entries all lie in the last 65534 ranks are
counted from 16-bit column distances (bitmaps and 16-bit tables in LDS), the
others from 32-bit columns. Graphs whose vertex counts straddle that limit,
rows of every work class on both sides of it, tasks of odd and even first and
last entries, and rows longer than an LDS hit counter holds are compared with
the oracle or closed forms (integers: tolerance 0)."""
from math import comb

import numpy as np
import pytest

import graphgen
import oracle
import smallgraphs as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda")


def check(tc, s, d, n):
    U = oracle.preprocess(s, d, n)
    T = oracle.count(U)
    w = oracle.wedges(U)
    g = tc.tc_preprocess(dev(s), dev(d), n)
    handles = [g] + [tc.tc_graph_retune(g, p) for p in (
        {"heavy_min": 0, "min_groups": 0}, {"pack_slots": 1024, "pack_target": 1024, "wave_chunk": 1024})]
    for h in handles:
        info = h.info()
        assert (info["probes"], info["tasks"]) == (w["probes"], w["tasks"])
        assert sum(c["probes"] for c in tc.tc_graph_class_stats(h).values()) == w["probes"]
        assert int(tc.tc_count(h).item()) == T
        for mode in (oracle.MODE_FULL, oracle.MODE_ORIENTED):
            want = oracle.support(U, mode)[1]
            assert np.array_equal(tc.tc_edge_support(h, mode)[0].cpu().numpy(), want), mode
        assert np.array_equal(tc.tc_vertex_triangles(h).cpu().numpy(), oracle.vertex_triangles(U))
    for tuning in (None, {"lds_cap_log2": 6}):
        plan = tc.tc_batch_create(handles, tuning=tuning)
        assert tc.tc_batch_count(plan).tolist() == [T] * len(handles)
        plan.free()


# (the oracle's ranks are the graph's: a dense block on the ids that end up
# last and first gives both kinds of rows heavy work)
@pytest.mark.parametrize("n", [65533, 65534, 65535, 65536, 65600, 66001, 140001])
def test_vertex_counts_around_the_span(tc, n):
    rng = np.random.default_rng(n)
    s, d = graphgen.rmat(17, 6, seed=3)
    s, d = s % n, d % n  # hubs, and low rows with entries on both sides of the limit
    k = 300
    iu = np.triu_indices(k, 1)
    low = rng.permutation(n)[:k].astype(np.int32)
    print("case n=%d" % n, flush=True)
    check(tc, np.concatenate([s, low[iu[0]]]), np.concatenate([d, low[iu[1]]]), n)


def test_long_rows_below_the_span(tc):
    # 40 vertices of degree 50000 over a ring: low rows (the ring's) reach
    # across the limit, the hubs' rows are short ones
    n = 70000
    hubs = np.repeat(np.arange(40), 50000)
    s = np.concatenate([hubs, np.arange(n)])
    d = np.concatenate([np.tile(np.arange(100, 50100), 40), (np.arange(n) + 1) % n])
    check(tc, s.astype(np.int32), d.astype(np.int32), n)


def test_rows_longer_than_the_hit_counters(tc):
    # K_n with rows of more than 8192 keys: FULL support credits their (b, k)
    # edges one by one; every edge lies in n - 2 triangles
    n = 8200
    iu = np.triu_indices(n, 1)
    g = tc.tc_preprocess(dev(iu[0]), dev(iu[1]), n)
    assert int(tc.tc_count(g).item()) == comb(n, 3)
    sup, _ = tc.tc_edge_support(g, tc.TC_SUPPORT_FULL)
    assert int(sup.min().item()) == int(sup.max().item()) == n - 2
    t = tc.tc_vertex_triangles(g)
    assert int(t.min().item()) == int(t.max().item()) == comb(n - 1, 2)


@pytest.mark.parametrize("case", ["star", "path", "one_edge", "K3", "K5_in_65540"])
def test_smallest(tc, case):
    if case == "K5_in_65540":  # two ranks outside the span, the K5 at its end
        s, d, n = sg.complete(5)
        n = 65540
    else:
        s, d, n = {"star": sg.star(9), "path": (np.arange(5), np.arange(1, 6), 6),
                   "one_edge": (np.array([0]), np.array([1]), 2), "K3": sg.complete(3)}[case]
    check(tc, np.asarray(s, np.int32), np.asarray(d, np.int32), n)
