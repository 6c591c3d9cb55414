"""The k-truss peel's list of work entries: every number of entries per edge,
at walks of just under, at and over a chunk, against the oracle and closed
forms (integers: tolerance 0); what the list takes of the card's memory."""
import gc

import numpy as np
import pytest

import graphgen
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


def build(tc, s, d, n):
    return tc.tc_preprocess(*(torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to("cuda") for x in (s, d)), n)


@pytest.mark.parametrize("walks", ["16", "8", "4", "2", "1"])
def test_entries_per_edge(tc, monkeypatch, walks):
    monkeypatch.setenv("TC_TRUSS_WALKS", walks)
    for n in (65, 66, 129, 257, 513, 1025, 1100):
        print("case walks=%s n=%d" % (walks, n), flush=True)
        iu = np.triu_indices(n, 1)
        keep = np.ones(iu[0].size, bool)
        keep[::n] = False  # several levels, and rounds that walk
        s, d = iu[0][keep], iu[1][keep]
        U = oracle.preprocess(s.astype(np.int32), d.astype(np.int32), n) if n < 600 else None
        g = build(tc, s, d, n)
        tau, kmax = tc.tc_truss(g)
        if U is not None:
            want_k, want = oracle.truss(U)
            assert np.array_equal(tau.cpu().numpy(), want) and kmax == want_k
        else:  # the same as with whole walks
            monkeypatch.setenv("TC_TRUSS_WALKS", "1")
            tau1, kmax1 = tc.tc_truss(g)
            monkeypatch.setenv("TC_TRUSS_WALKS", walks)
            assert torch.equal(tau, tau1) and kmax == kmax1
    s, d = graphgen.rmat(12, seed=3)
    hub = np.arange(1, 1 << 12)
    s, d = np.concatenate([s, np.zeros_like(hub)]), np.concatenate([d, hub])
    U = oracle.preprocess(s.astype(np.int32), d.astype(np.int32), 1 << 12)
    want_k, want = oracle.truss(U)
    tau, kmax = tc.tc_truss(build(tc, s, d, 1 << 12))
    assert np.array_equal(tau.cpu().numpy(), want) and kmax == want_k


def test_list_bytes(tc):
    # a complete graph of 1025 vertices takes the most entries, 16 of 8 bytes an
    # edge; the call's blocks (rounded up by at most 2 MiB each) stay in the
    # library's cache
    n = 1025
    iu = np.triu_indices(n, 1)
    g = build(tc, iu[0], iu[1], n)
    tau = torch.empty(g.m, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    gc.collect()
    tc.tc_release_cached_memory()
    assert tc.tc_memory_stats()["cached"] == 0
    kmax = tc.tc_truss(g, tau)[1]
    assert kmax == n
    held = tc.tc_memory_stats()["cached"]
    assert held <= (44 + 128) * g.m + 8 * n + 20 * (2 << 20), (held, g.m)
