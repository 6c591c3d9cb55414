"""k-truss peels of no, one, a few and many rounds: equal supports are answered
without a peel, the host reads back once per 32 rounds, and the last edges'
frontier is not walked. Against the oracle."""
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
    s, d = (np.ascontiguousarray(x, dtype=np.int32) for x in (s, d))
    U = oracle.preprocess(s, d, n)
    want_k, want = oracle.truss(U)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    tau, kmax = tc.tc_truss(g)
    assert np.array_equal(tau.cpu().numpy(), want) and kmax == want_k


@pytest.mark.parametrize("n", [4, 6, 8, 9, 10, 12, 20, 40, 42, 44, 46, 60, 100, 104, 105, 200, 300])
def test_square_of_a_path(tc, n):
    # one level; a round takes what the two ends have left: about n / 2 rounds
    v = np.arange(n)
    print("case n=%d" % n, flush=True)
    check(tc, np.concatenate([v[:-1], v[:-2]]), np.concatenate([v[1:], v[2:]]), n)


@pytest.mark.parametrize("levels", [1, 2, 3, 5, 9, 17, 30])
def test_cliques_of_every_size(tc, levels):
    # disjoint cliques of 2, 3, ... vertices: every level is one round
    s, d, at = [], [], 0
    for k in range(2, levels + 2):
        i = np.triu_indices(k, 1)
        s.append(at + i[0])
        d.append(at + i[1])
        at += k
    print("case levels=%d" % levels, flush=True)
    check(tc, np.concatenate(s), np.concatenate(d), at)


@pytest.mark.parametrize("case", ["edge", "path", "star", "triangle", "two_cliques", "clique_and_edge", "bipartite"])
def test_equal_supports(tc, case):
    k5 = np.triu_indices(5, 1)
    s, d, n = {"edge": ([0], [1], 2), "path": (np.arange(70), np.arange(1, 71), 71),
               "star": (np.zeros(99), np.arange(1, 100), 100), "triangle": ([0, 1, 2], [1, 2, 0], 3),
               "two_cliques": (np.concatenate([k5[0], k5[0] + 5]), np.concatenate([k5[1], k5[1] + 5]), 10),
               "clique_and_edge": (np.append(k5[0], 5), np.append(k5[1], 6), 7),
               "bipartite": (np.repeat(np.arange(20), 30), np.tile(np.arange(20, 50), 20), 50)}[case]
    print("case %s" % case, flush=True)
    check(tc, np.asarray(s), np.asarray(d), n)


@pytest.mark.parametrize("n,p", [(80, 0.99), (120, 0.5), (400, 0.9), (500, 0.05)])
def test_dense(tc, n, p):
    i = np.triu_indices(n, 1)
    keep = np.random.default_rng(n).random(i[0].size) < p
    print("case n=%d p=%.2f" % (n, p), flush=True)
    check(tc, i[0][keep], i[1][keep], n)
