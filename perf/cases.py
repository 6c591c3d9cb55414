"""Timing cases of the framework: what its users run, over the sizes they run it at.

Every case is one call sequence through the public entry points on seeded
synthetic graphs: RMAT (0.57, 0.19, 0.19, 0.05) with scrambled ids - the shape
of the Graph500 inputs - or Erdos-Renyi pairs, as raw pairs with duplicates
and self loops. Kinds ("kind" of a case):

  step        raw pairs in HBM -> tc_preprocess -> tc_count (-> tc_graph_export): the whole path of one graph
  count       tc_count on a resident graph
  support     tc_edge_support (full or oriented) on a resident graph
  block       tc_block_count: one rank of the q x q cyclic grid, with its per-shift counts
  batch       tc_batch_count of a planned batch of uneven graphs
  clustering  tc_clustering with the per-vertex triangles and the two sums
  truss       tc_truss of every edge
  serve       a burst of host edge lists through a running Server, counts and full supports mixed

All results are whole numbers except the clustering coefficients (float64).
"""
import math
import random

import numpy as np
import torch

import paper_1907_09575_amd as tc

_QUADRANTS = (0.57, 0.76, 0.95)  # cumulative a, a + b, a + b + c


def listed():
    return [
        # the smallest call of the framework's own configurations: launches and host latency
        {"name": "step_er_4096", "kind": "step", "model": "er", "n": 4096, "pairs": 32768, "export": False},
        # a sparse graph with even degrees at odd sizes, whose U the caller takes out
        {"name": "step_er_odd", "kind": "step", "model": "er", "n": 1000003, "pairs": 8000021, "export": True},
        # an everyday power-law graph from raw pairs to its count
        {"name": "step_rmat20", "kind": "step", "model": "rmat", "n": 1 << 20, "pairs": 16 << 20, "export": False},
        # the headline: RMAT scale 24, edge factor 16, raw pairs to the count
        {"name": "step_rmat24", "kind": "step", "model": "rmat", "n": 1 << 24, "pairs": 16 << 24, "export": False},
        # counting again on a graph that stays resident
        {"name": "count_rmat22", "kind": "count", "model": "rmat", "n": 1 << 22, "pairs": 16 << 22},
        # per-edge support, both modes; the oriented one at odd sizes
        {"name": "full_rmat20", "kind": "support", "model": "rmat", "n": 1 << 20, "pairs": 16 << 20, "full": True},
        {"name": "oriented_rmat_odd", "kind": "support", "model": "rmat", "n": 700001, "pairs": 11200003, "full": False},
        # one rank of the 13 x 13 grid of the headline graph
        {"name": "block_rmat24_q13", "kind": "block", "model": "rmat", "n": 1 << 24, "pairs": 16 << 24, "q": 13, "x": 0, "y": 0},
        # many small uneven graphs in one launch
        {"name": "batch_512", "kind": "batch", "graphs": 512},
        # uses of the counts
        {"name": "clustering_rmat20", "kind": "clustering", "model": "rmat", "n": 1 << 20, "pairs": 16 << 20},
        {"name": "truss_rmat18", "kind": "truss", "model": "rmat", "n": 1 << 18, "pairs": 16 << 18},
        # requests of a server, median 2^14 vertices
        {"name": "serve_64", "kind": "serve", "requests": 64},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# smallest and largest number of vertices of a drawn graph, by kind
_RANGES = {"step": (64, 1 << 23), "count": (256, 1 << 22), "support": (256, 1 << 20), "block": (1 << 14, 1 << 23),
           "clustering": (256, 1 << 20), "truss": (256, 1 << 18)}


def draw(rng):
    """One more case: kinds by weight, sizes over the logarithm of their range, odd ones among them."""
    kind = rng.choice(["step"] * 4 + ["count"] * 2 + ["support"] * 3 + ["block", "batch", "clustering", "truss", "serve"])
    if kind == "batch":
        return {"kind": "batch", "graphs": _log_int(rng, 16, 512)}
    if kind == "serve":
        return {"kind": "serve", "requests": _log_int(rng, 4, 64)}
    lo, hi = _RANGES[kind]
    n = _log_int(rng, lo, hi)
    c = {"kind": kind, "model": rng.choice(["rmat", "rmat", "er"]), "n": n, "pairs": int(n * rng.uniform(4, 24))}
    if kind == "step":
        c["export"] = rng.random() < 0.3
    elif kind == "support":
        c["full"] = rng.random() < 0.5
    elif kind == "block":
        c["q"] = rng.randint(2, 16)
        c["x"], c["y"] = rng.randrange(c["q"]), rng.randrange(c["q"])
    return c


# ---- inputs ------------------------------------------------------------------


def _pairs(model, n, m, gen):
    """m raw pairs over n vertices as two int32 tensors on the GPU."""
    dev = gen.device
    if model == "er":
        return (torch.randint(0, n, (m,), device=dev, dtype=torch.int32, generator=gen),
                torch.randint(0, n, (m,), device=dev, dtype=torch.int32, generator=gen))
    ab, abc = _QUADRANTS[1], _QUADRANTS[2]
    src = torch.zeros(m, dtype=torch.int32, device=dev)
    dst = torch.zeros(m, dtype=torch.int32, device=dev)
    for _ in range(max(1, (n - 1).bit_length())):
        r = torch.rand(m, device=dev, generator=gen)
        down = r >= ab
        right = (r >= _QUADRANTS[0]) & ~down | (r >= abc)
        src.mul_(2).add_(down)
        dst.mul_(2).add_(right)
    ids = torch.randperm(n, device=dev, generator=gen).to(torch.int32)  # scrambled ids
    return ids[src.remainder_(n)], ids[dst.remainder_(n)]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _many(case):
    """(model, n, pairs) of the graphs of a batch or a burst."""
    rng = random.Random(17)
    out = []
    if case["kind"] == "batch":  # n log-uniform in [64, 65536]; even index ER, odd index RMAT
        for g in range(case["graphs"]):
            n = _log_int(rng, 64, 65536)
            out.append(("er", n, int(n * rng.uniform(8, 64) / 2)) if g % 2 == 0 else ("rmat", n, int(n * rng.uniform(8, 32))))
    else:  # ln n normal around 2^14
        for _ in range(case["requests"]):
            n = int(min(1 << 18, max(64, round(math.exp(rng.gauss(math.log(1 << 14), 1.0))))))
            out.append(("er", n, 8 * n) if rng.random() < 0.5 else ("rmat", n, 16 * n))
    return out


def prepare(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind == "batch":
        graphs = [tc.tc_preprocess(*_pairs(model, n, m, gen), n) for model, n, m in _many(case)]
        return {"case": case, "plan": tc.tc_batch_create(graphs),
                "counts": torch.empty(len(graphs), dtype=torch.int64, device="cuda")}
    if kind == "serve":
        reqs = []
        for i, (model, n, m) in enumerate(_many(case)):
            src, dst = (t.cpu().numpy() for t in _pairs(model, n, m, gen))
            full = i % 2 == 1
            reqs.append(("support" if full else "count", src, dst, n, np.zeros(m, dtype=np.int32) if full else None))
        return {"case": case, "reqs": reqs, "server": tc.Server(32 << 30, max_slots=64, options={"prep_threads": 8})}
    src, dst = _pairs(case["model"], case["n"], case["pairs"], gen)
    # per-edge outputs have room for one value per raw pair (the simple graph
    # has at most that many edges; the rest stays 0)
    if kind == "step":
        st = {"case": case, "src": src, "dst": dst}
        if case["export"]:
            st["row_ptr"] = torch.empty(case["n"] + 1, dtype=torch.int64, device="cuda")
            st["col"] = torch.zeros(case["pairs"], dtype=torch.int32, device="cuda")
            st["perm"] = torch.empty(case["n"], dtype=torch.int32, device="cuda")
        return st
    st = {"case": case, "graph": tc.tc_preprocess(src, dst, case["n"])}
    if kind == "count":
        st["count"] = torch.empty(1, dtype=torch.int64, device="cuda")
    elif kind == "support":
        st["count"] = torch.empty(1, dtype=torch.int64, device="cuda")
        st["support"] = torch.zeros(case["pairs"], dtype=torch.int32, device="cuda")
    elif kind == "block":
        st["count"] = torch.empty(1, dtype=torch.int64, device="cuda")
        st["per_shift"] = torch.empty(case["q"], dtype=torch.int64, device="cuda")
    elif kind == "clustering":
        st["cc"] = torch.empty(case["n"], dtype=torch.float64, device="cuda")
        st["tri"] = torch.empty(case["n"], dtype=torch.int64, device="cuda")
        st["sums"] = torch.empty(2, dtype=torch.int64, device="cuda")
    elif kind == "truss":
        st["tau"] = torch.zeros(case["pairs"], dtype=torch.int32, device="cuda")
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        g = tc.tc_preprocess(state["src"], state["dst"], case["n"])
        count = tc.tc_count(g)
        out = [count, g.m]
        if case["export"]:
            tc.tc_graph_export(g, row_ptr=state["row_ptr"], col=state["col"], perm=state["perm"])
            out += [state["row_ptr"], state["col"], state["perm"]]
        tc.tc_graph_free(g)
        return out
    if kind == "count":
        return tc.tc_count(state["graph"], out=state["count"])
    if kind == "support":
        mode = tc.TC_SUPPORT_FULL if case["full"] else tc.TC_SUPPORT_ORIENTED
        tc.tc_edge_support(state["graph"], mode, support=state["support"], count=state["count"])
        return [state["support"], state["count"]]
    if kind == "block":
        return list(tc.tc_block_count(state["graph"], case["q"], case["x"], case["y"], count=state["count"],
                                      per_shift=state["per_shift"]))
    if kind == "batch":
        return tc.tc_batch_count(state["plan"], state["counts"])
    if kind == "clustering":
        return list(tc.tc_clustering(state["graph"], cc=state["cc"], tri=state["tri"], sums=state["sums"]))
    if kind == "truss":
        return [state["tau"], tc.tc_truss(state["graph"], tau=state["tau"])[1]]
    server = state["server"]
    tickets = [server.submit(op, src, dst, n, support_out=sup) for op, src, dst, n, sup in state["reqs"]]
    results = [server.poll(t) for t in tickets]
    return [np.array([r["count"] for r in results], dtype=np.int64)] + [r[4] for r in state["reqs"] if r[4] is not None]


def work(case):
    """Bytes of the inputs and outputs, each moved once (the lookups of the
    intersections depend on the graph drawn and are not counted; no floating
    point work to speak of)."""
    kind = case["kind"]
    if kind == "batch":  # row pointers and columns of each graph, and its count
        return {"bytes": sum(8 * n + 4 * m + 8 for _, n, m in _many(case)), "flops": 0}
    if kind == "serve":  # raw pairs in, a support per edge out for every second request
        return {"bytes": sum(8 * m + (4 * m if i % 2 else 0) + 8 for i, (_, _, m) in enumerate(_many(case))), "flops": 0}
    n, m = case["n"], case["pairs"]
    if kind == "step":
        return {"bytes": 8 * m + 8 + ((12 * n + 4 * m) if case["export"] else 0), "flops": 0}
    resident = 8 * n + 4 * m
    if kind == "block":  # the rank's hashed and probed rows
        return {"bytes": 2 * resident // case["q"] + 8 * case["q"], "flops": 0}
    out = {"count": 8, "support": 4 * m + 8, "clustering": 16 * n + 16, "truss": 4 * m + 4}[kind]
    return {"bytes": resident + out, "flops": 0}


# ---- the same results from torch alone -----------------------------------------

_WEDGES_MAX = 6 << 30  # lookups above which exact() would take too long


def _padded(x, size):
    return torch.nn.functional.pad(x, (0, size - x.numel()))


def _simple(src, dst, n):
    """Degree-ordered upper triangle of the simple graph of raw pairs:
    row_ptr, col, perm (rank of every vertex), sorted keys row * n + col, degrees."""
    u, v = src.to(torch.int64), dst.to(torch.int64)
    key = torch.unique((torch.minimum(u, v) * n + torch.maximum(u, v))[u != v])
    lo, hi = key // n, key % n
    deg = torch.bincount(lo, minlength=n) + torch.bincount(hi, minlength=n)
    order = torch.argsort(deg * n + torch.arange(n, device=key.device))
    perm = torch.empty_like(order)
    perm[order] = torch.arange(n, device=key.device)
    a, b = perm[lo], perm[hi]
    okey = torch.sort(torch.minimum(a, b) * n + torch.maximum(a, b)).values
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=key.device)
    torch.cumsum(torch.bincount(okey // n, minlength=n), 0, out=row_ptr[1:])
    return row_ptr, okey % n, perm, okey, deg


def _triangles(row_ptr, col, okey, n):
    """Triangles a < b < k as U positions of their edges (a, b), (a, k), (b, k),
    a chunk of tasks at a time."""
    m = col.numel()
    if m == 0:
        return
    i = torch.arange(m, device=col.device)
    length = row_ptr[okey // n + 1] - i - 1
    ends = torch.cumsum(length, 0)
    start = 0
    while start < m:
        base = int(ends[start - 1]) if start else 0
        stop = max(start + 1, int(torch.searchsorted(ends, base + (1 << 26), right=True)))
        e = torch.repeat_interleave(i[start:stop], length[start:stop])
        off = torch.arange(e.numel(), device=col.device) - (ends[e] - length[e] - base)
        p = e + 1 + off
        want = col[e] * n + col[p]
        at = torch.searchsorted(okey, want).clamp_(max=m - 1)
        hit = okey[at] == want
        yield e[hit], p[hit], at[hit]
        start = stop


def _wedges(row_ptr):
    d = row_ptr[1:] - row_ptr[:-1]
    return int((d * (d - 1) // 2).sum())


def _count(row_ptr, col, okey, n):
    return sum(int(e.numel()) for e, _, _ in _triangles(row_ptr, col, okey, n))


def _support(row_ptr, col, okey, n, full):
    s = torch.zeros(col.numel(), dtype=torch.int64, device=col.device)
    for edges in _triangles(row_ptr, col, okey, n):
        for x in edges if full else edges[:1]:
            s += torch.bincount(x, minlength=col.numel())
    return s


def _trussness(row_ptr, col, okey, n):
    """Peeling over the list of all triangles."""
    m = col.numel()
    tau = torch.zeros(m, dtype=torch.int64, device=col.device)
    if m == 0:
        return tau, 0
    tri = torch.cat([torch.stack(t).to(torch.int32) for t in _triangles(row_ptr, col, okey, n)], 1)
    sup = torch.zeros(m, dtype=torch.int64, device=col.device)
    for x in tri:
        sup += torch.bincount(x, minlength=m)
    alive = torch.ones(m, dtype=torch.bool, device=col.device)
    k = 3
    while True:
        left = sup[alive]
        if left.numel() == 0:
            return tau, int(tau.max())
        k = max(k, int(left.min()) + 3)
        gone = alive & (sup < k - 2)
        if not bool(gone.any()):
            k += 1
            continue
        tau[gone] = k - 1
        alive &= ~gone
        dead = gone[tri[0]] | gone[tri[1]] | gone[tri[2]]
        for x in tri[:, dead]:
            sup -= torch.bincount(x, minlength=m)
        tri = tri[:, ~dead]


def exact(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind in ("batch", "serve"):
        counts, supports = [], []
        for i, (model, n, m) in enumerate(_many(case)):
            row_ptr, col, _, okey, _ = _simple(*_pairs(model, n, m, gen), n)
            if kind == "serve" and i % 2 == 1:
                s = _support(row_ptr, col, okey, n, True)
                supports.append(_padded(s, m))
                counts.append(int(s.sum()) // 3)
            else:
                counts.append(_count(row_ptr, col, okey, n))
        counts = torch.tensor(counts, dtype=torch.int64)
        return counts if kind == "batch" else [counts] + supports
    n = case["n"]
    if case["pairs"] > 1 << 27:
        return None
    row_ptr, col, perm, okey, deg = _simple(*_pairs(case["model"], n, case["pairs"], gen), n)
    if _wedges(row_ptr) > _WEDGES_MAX:
        return None
    if kind == "step":
        out = [_count(row_ptr, col, okey, n), int(col.numel())]
        return out + [row_ptr, _padded(col, case["pairs"]), perm] if case["export"] else out
    if kind == "count":
        return _count(row_ptr, col, okey, n)
    if kind == "support":
        s = _support(row_ptr, col, okey, n, case["full"])
        return [_padded(s, case["pairs"]), int(s.sum()) // (3 if case["full"] else 1)]
    if kind == "block":
        q, x, y = case["q"], case["x"], case["y"]
        per = torch.zeros(q, dtype=torch.int64, device=col.device)
        for e, p, _ in _triangles(row_ptr, col, okey, n):
            mine = (col[e] % q == x) & ((okey[e] // n) % q == y)
            per += torch.bincount((col[p][mine] - x - y) % q, minlength=q)
        return [per.sum(), per]
    if kind == "clustering":
        t = torch.zeros(n, dtype=torch.int64, device=col.device)
        for e, p, _ in _triangles(row_ptr, col, okey, n):
            for v in (okey[e] // n, col[e], col[p]):
                t += torch.bincount(v, minlength=n)
        pairs = deg * (deg - 1) // 2
        t = t[perm]
        cc = torch.where(pairs > 0, t.double() / pairs.clamp(min=1).double(), torch.zeros((), dtype=torch.float64, device=t.device))
        return [cc, t, torch.stack([t.sum(), pairs.sum()])]
    if _wedges(row_ptr) > 1 << 29:
        return None
    tau, kmax = _trussness(row_ptr, col, okey, n)
    return [_padded(tau, case["pairs"]), kmax]
