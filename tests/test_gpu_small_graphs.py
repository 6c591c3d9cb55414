"""The preprocessing of small graphs (at most 32768 vertices: one work-group
ranks and orders the rows; at most 16384 raw pairs: one work-group sorts them)
at the edges of its sizes, against the oracle: CSR, ranks, work counts, T and
full support, integer by integer."""
import numpy as np
import pytest

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


def check(tc, s, d, n):
    s, d = np.ascontiguousarray(s, dtype=np.int32), np.ascontiguousarray(d, dtype=np.int32)
    U = oracle.preprocess(s, d, n)
    T = oracle.count(U)
    w = oracle.wedges(U)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    rp, col, perm = tc.tc_graph_export(g)
    assert np.array_equal(perm.cpu().numpy(), U.rank)
    assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
    assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
    info = g.info()
    assert (info["probes"], info["tasks"], info["wedges_plus"]) == (w["probes"], w["tasks"], w["wedges_plus"])
    cls = tc.tc_graph_class_stats(g)
    assert sum(c["probes"] for c in cls.values()) == w["probes"]
    assert sum(c["tasks"] for c in cls.values()) == w["tasks"]
    assert int(tc.tc_count(g).item()) == T
    full = tc.tc_edge_support(g, tc.TC_SUPPORT_FULL)[0].cpu().numpy()
    assert np.array_equal(full, oracle.support(U, oracle.MODE_FULL)[1][:U.m])
    for p in ({"pack_target": 1024, "pack_slots": 1024, "wave_chunk": 1024}, {"heavy_min": 0}):
        h = tc.tc_graph_retune(g, p)
        assert int(tc.tc_count(h).item()) == T


def skewed(n, m, seed):
    # ids with a heavy head, duplicates and self loops among them
    rng = np.random.default_rng(seed)
    f = lambda: np.minimum((n * rng.random(m) ** 3).astype(np.int64), n - 1)
    return f(), f()


@pytest.mark.parametrize("n", [3, 255, 256, 257, 1023, 1025, 4096, 8191, 16383, 16384, 16385, 32767, 32768, 32769])
def test_vertex_counts(tc, n):
    print("case n=%d" % n, flush=True)
    check(tc, *skewed(n, 12 * n, n), n)


@pytest.mark.parametrize("m", [1, 2, 64, 4095, 4096, 4097, 8192, 8193, 16383, 16384, 16385, 20000])
def test_raw_pair_counts(tc, m):
    print("case m=%d" % m, flush=True)
    check(tc, *skewed(1500, m, m), 1500)


@pytest.mark.parametrize("case", ["star64", "star4096", "K64", "K181", "empty", "loops", "one_vertex"])
def test_degrees_and_degenerate_inputs(tc, case):
    # star: a degree of n - 1 with n a power of two (all sorted degree bits set)
    if case.startswith("star"):
        n = int(case[4:])
        s, d = np.zeros(n - 1, np.int64), np.arange(1, n)
    elif case.startswith("K"):
        s, d, n = sg.complete(int(case[1:]))
    elif case == "empty":
        s, d, n = np.zeros(0, np.int64), np.zeros(0, np.int64), 700
    elif case == "loops":
        s, d, n = np.arange(50), np.arange(50), 50
    else:
        s, d, n = np.zeros(3, np.int64), np.zeros(3, np.int64), 1
    if case in ("empty", "loops", "one_vertex"):
        g = tc.tc_preprocess(torch.from_numpy(np.asarray(s, np.int32)).cuda(),
                             torch.from_numpy(np.asarray(d, np.int32)).cuda(), n)
        assert g.info()["m"] == 0 and int(tc.tc_count(g).item()) == 0
        assert np.array_equal(tc.tc_graph_export(g)[2].cpu().numpy(), np.arange(n))
    else:
        check(tc, s, d, n)


@pytest.mark.parametrize("m", [100, 30000])
def test_bad_ids(tc, m):
    s, d = skewed(1000, m, 5)
    for bad in (-1, 1000, 2 ** 31 - 1):
        t = s.copy()
        t[m // 2] = bad
        with pytest.raises(tc.TCError) as e:
            tc.tc_preprocess(torch.from_numpy(t.astype(np.int32)).cuda(), torch.from_numpy(d.astype(np.int32)).cuda(), 1000)
        assert e.value.status == 1
