"""tc_graph_class_stats against the row classes worked out from U: rows, keys,
tasks and probes of every class, and the work-groups that count it (short rows'
items are dealt to work-groups in bundles of equal weight)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CLASSES = ("pack_small", "pack_large", "wg_small", "wg_large", "wg_huge", "wg_giant", "global")


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


def log2_up(x):
    return max(0, int(x - 1).bit_length())


def expected(U, heavy_min=2048):
    """Per class: rows, keys, tasks, probes, units (pairs of column entries)."""
    deg = np.diff(U.row_ptr)
    out = {c: [0, 0, 0, 0, 0] for c in CLASSES}
    tasks, probes, units = (np.zeros(U.n, np.int64) for _ in range(3))
    rows = np.repeat(np.arange(U.n), deg)
    pos = np.arange(U.m)
    col, end = U.col[:U.m], U.row_ptr[rows + 1]
    ok = (end - pos - 1 > 0) & (deg[col] > 0)
    first = pos + 1
    np.add.at(tasks, col[ok], 1)
    np.add.at(probes, col[ok], (end - first)[ok])
    np.add.at(units, col[ok], ((end + 1) // 2 - first // 2)[ok])
    for b in np.nonzero(units)[0]:
        d = int(deg[b])
        want = 4 * d if d <= 2048 else 2 * d
        l = 6 if want <= 64 else log2_up(want)
        c = ("global" if l > 14 else "wg_giant" if l > 13 else "wg_huge" if l > 12 else
             ("pack_small" if l <= 8 else "pack_large") if 2 * units[b] < heavy_min and l <= 10 else
             "wg_small" if l <= 10 else "wg_large")
        for i, v in enumerate((1, d, tasks[b], probes[b], units[b])):
            out[c][i] += int(v)
    return out


@pytest.mark.parametrize("case", ["skewed", "hubs", "clique"])
def test_short_rows(tc, case):
    rng = np.random.default_rng(11)
    if case == "clique":
        n = 700
        s, d = (x.astype(np.int32) for x in np.triu_indices(n, 1))
    else:
        n, m = (20000, 600000) if case == "skewed" else (30000, 300000)
        f = lambda: np.minimum((n * rng.random(m) ** 3).astype(np.int32), n - 1)
        s, d = f(), f()
        if case == "hubs":  # rows of more than 4096 keys: vertices that most of the others join to both ways
            far = np.arange(60, n, 3, dtype=np.int32)
            s = np.concatenate([s] + [np.full(far.size, h, np.int32) for h in range(12)])
            d = np.concatenate([d] + [far] * 12)
    U = oracle.preprocess(s, d, n)
    g = tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n)
    got = tc.tc_graph_class_stats(g)
    want = expected(U)
    heavy = 2 * sum(want[c][4] for c in CLASSES[2:])  # the bundles' weight, in probes
    least = max(4096, min(24 << 10, heavy // 2048))
    bundle = min(256 << 10, max(heavy // 16384, least))
    for c in CLASSES:
        st = got[c]
        assert (st["rows"], st["table_keys"], st["tasks"], st["probes"]) == tuple(want[c][:4]), c
        if c in CLASSES[2:]:
            assert st["workgroups"] == -(-want[c][4] // (bundle // 2)), (c, st["workgroups"])
        else:
            assert (st["workgroups"] > 0) == (want[c][0] > 0)
