"""The k-truss peel's work lists: neighbourhoods cut into several entries per
edge (more than 256 neighbours), frontiers that fill a wave's queue several
times, levels without rounds between them and long chains of rounds, against
closed forms and the oracle (integers: tolerance 0)."""
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


def truss(tc, s, d, n):
    g = tc.tc_preprocess(*(torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to("cuda") for x in (s, d)), n)
    tau, kmax = tc.tc_truss(g)
    return tau.cpu().numpy(), kmax


@pytest.mark.parametrize("n", [257, 258, 600, 2200])
def test_complete_graphs(tc, n):
    # one level that removes every edge; 2200: chunks of more than 256 neighbours
    iu = np.triu_indices(n, 1)
    tau, kmax = truss(tc, iu[0], iu[1], n)
    assert kmax == n and np.all(tau == n)


def test_chain_of_rounds(tc):
    # a strip of K4s, each sharing an edge with the next: an edge within one K4
    # has support 2, a shared one 4; all go at one level
    n, k = 802, 400
    i = 2 * np.arange(k)
    s = np.concatenate([i, i, i, i + 1, i + 1, i + 2])
    d = np.concatenate([i + 1, i + 2, i + 3, i + 2, i + 3, i + 3])
    tau, kmax = truss(tc, s, d, n)
    assert kmax == 4 and np.all(tau == 4)


def test_many_rounds_in_a_level(tc):
    # the square of a path: every edge lies in one or two triangles, and the
    # two ends' edges start what removes them all at one level
    n = 400
    v = np.arange(n)
    s, d = np.concatenate([v[:-1], v[:-2]]), np.concatenate([v[1:], v[2:]])
    tau, kmax = truss(tc, s, d, n)
    assert kmax == 3 and np.all(tau == 3)


@pytest.mark.parametrize("scale,seed", [(11, 4), (13, 9)])
def test_rmat_against_the_oracle(tc, scale, seed):
    s, d = graphgen.rmat(scale, seed=seed)
    hub = np.arange(1, 1 << scale)  # vertex 0 joined to all: walks of thousands on one side
    s, d = np.concatenate([s, np.zeros_like(hub)]), np.concatenate([d, hub])
    U = oracle.preprocess(s.astype(np.int32), d.astype(np.int32), 1 << scale)
    want_k, want = oracle.truss(U)
    tau, kmax = truss(tc, s, d, 1 << scale)
    assert np.array_equal(tau, want) and kmax == want_k
