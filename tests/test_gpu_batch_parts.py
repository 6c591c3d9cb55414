"""Batches of few graphs, whose packs of short rows are cut into parts and whose
bundles stay apart, up to as many as fill the GPU: counts and both supports (a
part adds its own hits) against the oracle. Cliques (packs and rows with work-groups of
their own), graphs of one pack, a graph without tasks, thresholds that make
packs small, and plans in both orders."""
import re

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


def clique(n):
    i = np.triu_indices(n, 1)
    return i[0].astype(np.int32), i[1].astype(np.int32), n


def skewed(n, m):
    rng = np.random.default_rng(n + m)
    f = lambda: np.minimum((n * rng.random(m) ** 2).astype(np.int32), n - 1)
    return f(), f(), n


def sets():
    return {"one_small": [skewed(40, 300)], "one": [skewed(1000, 16000)], "clique": [clique(100)],
            "cliques": [clique(k) for k in (3, 17, 64, 100, 150, 400)],
            "none": [(np.array([0], np.int32), np.array([1], np.int32), 3)],
            "mixed": [skewed(50 + 37 * i, 400 + 900 * i) for i in range(12)] + [clique(120), (np.array([0], np.int32), np.array([0], np.int32), 2)],
            "large": [skewed(70000, 600000), clique(90)],
            "many": [clique(30 + i % 60) for i in range(300)]}


@pytest.mark.parametrize("name", sorted(sets()))
def test_counts_and_supports(tc, name):
    graphs = sets()[name]
    print("case %s" % name, flush=True)
    Us = [oracle.preprocess(s, d, n) for s, d, n in graphs]
    want = [oracle.count(U) for U in Us]
    gs = [tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n) for s, d, n in graphs]
    for tuning in (None, {"order": "input", "graph": 0}, {"pack_slots": 1024, "pack_target": 4096}, {"lds_cap_log2": 6}):
        P = tc.tc_batch_create(gs, tuning)
        for _ in range(2):
            assert tc.tc_batch_count(P).cpu().tolist() == want, tuning
        P.free()
    assert tc.tc_count_batched(gs).cpu().tolist() == want
    counts = torch.empty(len(gs), dtype=torch.int64, device="cuda")
    tc.tc_count_batched_noalloc(gs, counts)
    assert counts.cpu().tolist() == want
    # the support modes run through the server's plans
    if len(graphs) <= 16:
        with tc.Server(8 << 30, 32) as srv:
            for op, mode in (("support_full", oracle.MODE_FULL), ("support_oriented", oracle.MODE_ORIENTED)):
                tickets = [srv.submit(op, s, d, n) for s, d, n in graphs]
                for t, U, T in zip(tickets, Us, want):
                    r = srv.poll(t)
                    assert r["status"] == 0 and r["count"] == T and r["m"] == U.m
                    assert np.array_equal(np.asarray(r["support"])[:U.m], oracle.support(U, mode)[1][:U.m])


def test_noalloc_takes_the_fewest_units_at_its_limit(tc):
    """Near the end of the scratch array the units are as few as in a batch that
    needs no filling: a small plan's finer units do not make it a refusal."""
    med_raw = clique(300)
    med, tiny = (tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
                 for s, d, n in (med_raw, clique(3)))
    want = oracle.count(oracle.preprocess(*med_raw))
    K = 2

    def units(gs):
        P = tc.tc_batch_create(gs)
        u = tc.tc_batch_describe(P)["units"]
        P.free()
        return u

    # 65536 probes a unit and no cuts from 33.5 M probes on: far less than 100 of these graphs
    u_med, rest = divmod(units([med] * 100), 100)
    assert rest == 0 and units([tiny]) == 1
    assert units([med] * K) >= K * u_med + 64  # (finer where nothing else runs)

    def refusal(n_tiny):
        gs = [med] * K + [tiny] * n_tiny
        with pytest.raises(tc.TCError, match="bytes of scratch") as e:
            tc.tc_count_batched_noalloc(gs, torch.empty(len(gs), dtype=torch.int64, device="cuda"))
        needs, n_units = re.search(r"needs (\d+) bytes of scratch \((\d+) work units\)", str(e.value)).groups()
        return int(needs), int(n_units)

    n0 = 200000
    needs, n_units = refusal(n0)
    assert n_units == K * u_med + n0
    per = (refusal(2 * n0)[0] - needs) / n0
    n1 = n0 - int(np.ceil((needs - (64 << 20) + 512) / per))  # the most that fit (the arrays' ends are rounded up to 256)
    counts = torch.empty(K + n1, dtype=torch.int64, device="cuda")
    tc.tc_count_batched_noalloc([med] * K + [tiny] * n1, counts)
    assert counts.cpu().tolist() == [want] * K + [1] * n1
    refusal(n1 + 16)
    med.free()
    tiny.free()
