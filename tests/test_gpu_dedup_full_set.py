"""A group of more keys than the dedup's hash set holds: edges chosen so that
their mixed keys agree in the sort's top bits (one interval of 512 lower
endpoints, one value of the mix's top byte). The call sorts by all bits
instead. Against the oracle: CSR, ranks and T."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [9000, 16300, 20000, 60000])
def test_one_group(count):
    print("case count=%d" % count, flush=True)
    import paper_1907_09575_amd as tc
    n, s, low = 65537, 17, 9
    lo = np.repeat(np.arange(512, dtype=np.uint32), n)
    hi = np.tile(np.arange(n, dtype=np.uint32), 512)
    x = (hi * np.uint32(0x9E3779B1) + lo * np.uint32(0x6A09E667)) & np.uint32((1 << s) - 1)
    at = np.flatnonzero((hi > lo) & (x >> low == 37))[:count]
    assert at.size == count
    rng = np.random.default_rng(count)
    a, b = lo[at].astype(np.int32), hi[at].astype(np.int32)
    e = rng.integers(0, n, (2, 30000)).astype(np.int32)
    src, dst = np.concatenate([a, e[0], b[:500]]), np.concatenate([b, e[1], a[:500]])
    order = rng.permutation(src.size)
    src, dst = np.ascontiguousarray(src[order]), np.ascontiguousarray(dst[order])
    U = oracle.preprocess(src, dst, n)
    g = tc.tc_preprocess(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n)
    rp, col, perm = tc.tc_graph_export(g)
    assert np.array_equal(perm.cpu().numpy(), U.rank)
    assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
    assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
    assert int(tc.tc_count(g).item()) == oracle.count(U)
