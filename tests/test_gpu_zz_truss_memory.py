"""tc_truss on a card with little memory left (collected late: it fills the
card): its list of work entries takes fewer entries per edge, and the call
succeeds."""
import gc

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1907_09575_amd as tc
    torch.cuda.set_device(0)
    return tc


def fill_device(keep_bytes):
    spare = torch.empty(keep_bytes, dtype=torch.uint8, device="cuda")
    held = []
    size = 1 << 30
    while size >= (16 << 20):
        try:
            held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            size //= 2
    del spare
    torch.cuda.empty_cache()
    return held


def test_coarser_walks_when_memory_is_short(tc):
    # complete graph of 3000 vertices, m = 4.5 M: 44 m bytes are 198 MB, one entry
    # per edge 36 MB, sixteen 576 MB
    n = 3000
    iu = np.triu_indices(n, 1)
    g = tc.tc_preprocess(torch.from_numpy(iu[0].astype(np.int32)).cuda(), torch.from_numpy(iu[1].astype(np.int32)).cuda(), n)
    tau = torch.empty(g.m, dtype=torch.int32, device="cuda")
    assert tc.tc_truss(g, tau)[1] == n  # (its kernels are loaded before the card is filled)
    torch.cuda.synchronize()
    gc.collect()
    tc.tc_release_cached_memory()
    torch.cuda.empty_cache()
    tau.zero_()
    held = fill_device(400 << 20)
    print("holding %.1f GiB" % (sum(h.numel() for h in held) / 2 ** 30), flush=True)
    try:
        kmax = tc.tc_truss(g, tau)[1]
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert kmax == n and bool((tau == n).all())
