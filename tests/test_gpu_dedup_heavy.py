"""Edges given very many times: groups of equal top bits that run far past a
tile, holding one heavy edge, several that take turns, or heavy ones among
thousands of others; both directions; just under and over the length that is
sorted by all bits instead. Against the oracle: CSR, ranks and T."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 50000  # 16-bit ids: keys of 8 bits of lo, 16 mixed, 8 of lo; sorted by the top 16


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


def same_group(count):
    # edges (lo, hi) whose keys agree in the 16 bits that the sort orders by
    lo = np.arange(512, 768, dtype=np.uint64)[:, None]
    hi = np.arange(1000, N, dtype=np.uint64)[None, :]
    mixed = (hi * np.uint64(0x9E3779B1) + (lo & np.uint64(255)) * np.uint64(0x6A09E667)) & np.uint64(0xFFFF)
    a, b = np.nonzero(mixed >> np.uint64(8) == 77)
    pick = np.random.default_rng(4).permutation(a.size)[:count]
    return (lo[a[pick], 0].astype(np.int32), hi[0, b[pick]].astype(np.int32))


def check(tc, s, d):
    s, d = np.ascontiguousarray(s, dtype=np.int32), np.ascontiguousarray(d, dtype=np.int32)
    U = oracle.preprocess(s, d, N)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), N)
    rp, col, perm = tc.tc_graph_export(g)
    assert g.m == U.m
    assert np.array_equal(perm.cpu().numpy(), U.rank)
    assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
    assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
    assert int(tc.tc_count(g).item()) == oracle.count(U)


@pytest.mark.parametrize("edges,copies", [(1, 4300), (1, 8400), (1, 300000), (2, 100000), (7, 30011), (64, 3000),
                                          (1500, 40), (5000, 9), (1, (1 << 20) - 4000), (1, (1 << 20) + 4200),
                                          (1, (1 << 17) - 4000), (1, (1 << 17) + 100), (3, 400000)])
@pytest.mark.parametrize("order", ["shuffled", "in_turn"])
def test_heavy_edges(tc, edges, copies, order):
    print("case edges=%d copies=%d %s" % (edges, copies, order), flush=True)
    lo, hi = same_group(edges)
    rng = np.random.default_rng(edges + copies)
    which = np.tile(np.arange(edges), copies) if order == "in_turn" else rng.integers(0, edges, edges * copies)
    flip = rng.random(which.size) < 0.5
    s, d = np.where(flip, hi[which], lo[which]), np.where(flip, lo[which], hi[which])
    f = lambda: np.minimum((N * rng.random(60000) ** 2).astype(np.int32), N - 1)
    check(tc, np.concatenate([f(), s]), np.concatenate([f(), d]))
