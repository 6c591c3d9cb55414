"""Per-vertex counts, clustering and transitivity on a stream that is being
captured: refused (status 3) with nothing recorded, and the capture goes on.
Transitivity itself against the oracle."""
import ctypes

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


def build(tc, scale=10):
    s, d = graphgen.rmat(scale, seed=2)
    n = 1 << scale
    return tc.tc_preprocess(torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda(), n), oracle.preprocess(s, d, n)


@pytest.mark.parametrize("call", ["transitivity", "vertex_triangles", "clustering"])
def test_refused_while_capturing(tc, call):
    g, _ = build(tc)
    tri = torch.empty(g.n, dtype=torch.int64, device="cuda")
    cc = torch.empty(g.n, dtype=torch.float64, device="cuda")
    sums = torch.empty(2, dtype=torch.int64, device="cuda")
    st = torch.cuda.Stream()
    run = {"transitivity": lambda: tc.tc_transitivity(g, stream=st),
           "vertex_triangles": lambda: tc.tc_vertex_triangles(g, tri, stream=st),
           "clustering": lambda: tc.tc_clustering(g, cc, tri, sums, stream=st)}[call]
    run()  # (blocks of the sizes it takes are in the library's cache)
    torch.cuda.synchronize()
    hip = tc._lib
    stream, graph, nodes = ctypes.c_void_p(st.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(99)
    assert hip.hipStreamBeginCapture(stream, 2) == 0  # (relaxed: other streams go on)
    with pytest.raises(tc.TCError) as e:
        run()
    assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    assert e.value.status == 3 and nodes.value == 0
    run()
    torch.cuda.synchronize()


@pytest.mark.parametrize("scale", [3, 8, 14])
def test_transitivity(tc, scale):
    g, U = build(tc, scale)
    lo, hi = np.repeat(np.arange(U.n), np.diff(U.row_ptr)), U.col[:U.m]
    deg = np.bincount(lo, minlength=U.n) + np.bincount(hi, minlength=U.n)
    pairs = int((deg * (deg - 1) // 2).sum())
    assert tc.tc_transitivity(g) == (3 * oracle.count(U) / pairs if pairs else 0.0)
