"""Scans whose look-back waits end at once (TC_SCAN_SPINS=0): a tile then adds
the elements before it itself. Every scan of the preprocessing, of a retuned
handle and of a block must give the same offsets. Against the oracle."""
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


@pytest.mark.parametrize("spins", ["0", "1"])
@pytest.mark.parametrize("n,m", [(5000, 60000), (40000, 500000), (200001, 1300001)])
def test_waits_that_end(tc, monkeypatch, spins, n, m):
    print("case n=%d m=%d spins=%s" % (n, m, spins), flush=True)
    rng = np.random.default_rng(n)
    s, d = (np.minimum((n * rng.random(m) ** 2).astype(np.int32), n - 1) for _ in range(2))
    U = oracle.preprocess(s, d, n)
    monkeypatch.setenv("TC_SCAN_SPINS", spins)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    rp, col, perm = tc.tc_graph_export(g)
    assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
    assert np.array_equal(col.cpu().numpy(), U.col[:U.m])
    T = oracle.count(U)
    assert int(tc.tc_count(g).item()) == T
    assert int(tc.tc_count(tc.tc_graph_retune(g, {"heavy_min": 1024, "pack_slots": 1024})).item()) == T
    count, _ = tc.tc_block_count(g, 2, 1, 0)
    assert int(count.item()) == oracle.block_count_one(U, 2, 1, 0)[0]
