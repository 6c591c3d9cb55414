"""Preprocessing of small graphs by several host threads at once, each on its
own stream: blocks of temporaries, cleared words and scan words of calls that
really overlap. A bounded number of calls, ended by the first that fails;
against the oracle's CSR, ranks and T."""
import threading

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

THREADS, CALLS = 4, 12


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


@pytest.mark.parametrize("sizes", ["block_sorts", "one_block", "past_it", "mixed"])
def test_threads(tc, sizes):
    cases = []
    for i in range(THREADS * CALLS):
        n, m = {"block_sorts": (100 + 211 * i, 1001 + 301 * i), "one_block": (900 + 613 * i, 16385 + 977 * i),
                "past_it": (900 + 613 * i, 65537 + 3001 * i), "mixed": (300 + 1400 * i, 3 + 3071 * i)}[sizes]
        rng = np.random.default_rng(i + n)
        f = lambda: np.minimum((n * rng.random(m) ** 2).astype(np.int32), n - 1)
        s, d = f(), f()
        U = oracle.preprocess(s, d, n)
        cases.append((n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), U, oracle.count(U)))
    torch.cuda.synchronize()
    failed, start = [], threading.Barrier(THREADS)

    def work(t):
        try:
            torch.cuda.set_device(0)
            st = torch.cuda.Stream()
            start.wait()
            for j in range(CALLS):
                if failed:
                    return
                n, s, d, U, T = cases[j * THREADS + t]
                rp, col, perm = (torch.empty(k, dtype=ty, device="cuda") for k, ty in
                                 ((n + 1, torch.int64), (max(U.m, 1), torch.int32), (n, torch.int32)))
                c = torch.empty(1, dtype=torch.int64, device="cuda")
                torch.cuda.current_stream().synchronize()
                g = tc.tc_preprocess(s, d, n, stream=st)
                tc.tc_count(g, out=c, stream=st)
                tc.tc_graph_export(g, rp, col[:g.m], perm, stream=st)
                st.synchronize()
                assert g.m == U.m and int(c.item()) == T
                assert np.array_equal(perm.cpu().numpy(), U.rank)
                assert np.array_equal(rp.cpu().numpy(), U.row_ptr)
                assert np.array_equal(col[:U.m].cpu().numpy(), U.col[:U.m])
                g.free()
        except BaseException as e:  # noqa: BLE001 (reported by the main thread)
            failed.append((t, e))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
