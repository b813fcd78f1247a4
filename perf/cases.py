"""Workloads of the library for timing: queue operations, single shortest-path
queries, batched, round-form and served queries, each through the package's
public calls.

A case is a dict of plain values. ``prepare`` builds its inputs on the GPU from
a seed (graph, weights, source, output buffers, and the workspace object a
program keeps), ``run`` is one pass, ``work`` the bytes and operations a pass
cannot do without, ``exact`` the same outputs from plain tensor operations in
64-bit integers. Graph families, sizes and weight rules are those of the
benchmark and the tests: 4-neighbour grids with weights 1..100, road-like
meshes with 1 % diagonal shortcuts, RMAT and uniform random graphs, the last
three with potential-shifted weights (some negative, no negative cycle).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_21826_amd as bq

INF = torch.iinfo(torch.int64).max
ONE_WAVE = {"wg_size": 64, "wg_count": 1}


def listed():
    return [
        # a short FIFO hand-over by one wave, in order (the smallest call)
        {"name": "fifo_small", "kind": "fifo", "capacity": 1024, "items": 700},
        # a large task list through the queue at the default launch: filled,
        # drained, and each task's worker result written to its place
        {"name": "tasks_1m", "kind": "tasks", "capacity": 1 << 20, "items": 1000003, "b": 0},
        # concurrent producers and consumers on a ring much smaller than the
        # item count, with the record of what was delivered
        {"name": "mixed_4m", "kind": "mixed", "capacity": 1 << 16, "ops": 1 << 22, "b": 16},
        # one query on a small graph: latency; the CSR is checked as a first
        # call on unknown data does
        {"name": "er2k_checked", "kind": "sssp", "family": "er", "n": 2000, "deg": 8,
         "launch": "default", "pred": True, "validate": True, "mark": False},
        # one query on a small mesh: latency over a deep shortest-path tree
        {"name": "grid64", "kind": "sssp", "family": "grid", "n": 64, "deg": 4,
         "launch": "default", "pred": True, "validate": False, "mark": False},
        # one ordinary query with the library's own launch shape
        {"name": "er200k", "kind": "sssp", "family": "er", "n": 200000, "deg": 8,
         "launch": "default", "pred": True, "validate": False, "mark": False},
        # the benchmark's headline query, at the launch it times
        {"name": "rmat20", "kind": "sssp", "family": "rmat", "n": 20, "deg": 16,
         "launch": "tuned", "pred": True, "validate": False, "mark": False},
        # one query on a large road-like mesh in bucket order, as the
        # benchmark runs it
        {"name": "road2048", "kind": "sssp", "family": "road", "n": 2048, "deg": 4,
         "launch": "buckets", "pred": True, "validate": False, "mark": False},
        # many random graphs of uneven size in one launch
        {"name": "batch_er256", "kind": "batch", "family": "er", "count": 256, "lo": 1000,
         "hi": 200000, "pred": True},
        # many sources on one shared power-law graph
        {"name": "batch_rmat20x64", "kind": "batch", "family": "rmat", "count": 64, "lo": 20,
         "hi": 20, "pred": True},
        # the round form over the edge queue
        {"name": "rounds_rmat18", "kind": "rounds", "family": "rmat", "n": 18, "deg": 16, "b": 0},
        # a request mix on the served form: resident graphs and uploads
        {"name": "served_48", "kind": "served", "requests": 48, "scale": 16, "side": 256,
         "n": 50000, "uploads": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fifo", "tasks", "mixed", "sssp", "sssp", "sssp", "sssp", "noalloc",
                       "batch", "batch", "rounds", "served"])
    if kind == "fifo":
        cap = 1 << rng.randint(6, 13)
        return {"kind": kind, "capacity": cap, "items": rng.randint(1, cap)}
    if kind == "tasks":
        cap = 1 << rng.randint(10, 22)
        return {"kind": kind, "capacity": cap, "items": _log_int(rng, cap // 8, cap),
                "b": rng.choice([0, 2, 8, 16])}
    if kind == "mixed":
        return {"kind": kind, "capacity": 1 << rng.randint(12, 20), "ops": 1 << rng.randint(16, 22),
                "b": rng.choice([1, 4, 16, 64])}
    if kind in ("sssp", "noalloc"):
        family = rng.choice(["er", "er", "rmat", "grid", "road"])
        deg, launch = 4, "default"
        if family == "er":
            n, deg = _log_int(rng, 100, 1000000), rng.randint(3, 16)
        elif family == "rmat":
            n, deg = rng.randint(9, 20), rng.choice([8, 16])
            launch = rng.choice(["default", "tuned"])
        else:
            n = _log_int(rng, 8, 300)
            if rng.random() < 0.5:
                n, launch = _log_int(rng, 64, 2000), "buckets"
        if kind == "noalloc":
            n = {"er": min(n, 150000), "rmat": min(n, 17), "grid": min(n, 300),
                 "road": min(n, 300)}[family]
            return {"kind": kind, "family": family, "n": n, "deg": deg, "launch": launch,
                    "pred": rng.random() < 0.8}
        # marking runs keep a negative cycle behind the last vertex
        mark = family == "er" and rng.random() < 0.2
        return {"kind": kind, "family": family, "n": n, "deg": deg, "launch": launch,
                "pred": rng.random() < 0.8, "validate": rng.random() < 0.2, "mark": mark}
    if kind == "batch":
        if rng.random() < 0.6:
            lo = _log_int(rng, 30, 20000)
            return {"kind": kind, "family": "er", "count": _log_int(rng, 4, 256), "lo": lo,
                    "hi": min(200000, lo * rng.randint(2, 60)), "pred": rng.random() < 0.8}
        scale = rng.randint(10, 18)
        return {"kind": kind, "family": "rmat", "count": _log_int(rng, 4, 64), "lo": scale,
                "hi": scale, "pred": rng.random() < 0.8}
    if kind == "rounds":
        family = rng.choice(["er", "rmat"])
        n = rng.randint(8, 19) if family == "rmat" else _log_int(rng, 100, 400000)
        return {"kind": kind, "family": family, "n": n, "deg": 16 if family == "rmat" else 8,
                "b": rng.choice([0, 0, 64])}
    return {"kind": "served", "requests": rng.randint(6, 48), "scale": rng.randint(11, 17),
            "side": rng.randint(40, 300), "n": _log_int(rng, 2000, 100000),
            "uploads": rng.randint(0, 6)}


# ---------------------------------------------------------------------------
# graphs: CSR on the GPU (int64 offsets, int32 columns and weights)
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _ints(g, lo, hi, size):
    return torch.randint(lo, hi, (size,), generator=g, device="cuda", dtype=torch.int64)


def _csr(n, s, d, w):
    s, order = torch.sort(s, stable=True)
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(s, minlength=n), 0, out=off[1:])
    return off, d[order].to(torch.int32), w[order].to(torch.int32)


def _shifted(g, n, s, d):
    """w0 + p(u) - p(v), w0 in 1..1000, p in 0..1000: no negative cycle."""
    p = _ints(g, 0, 1001, n)
    return _ints(g, 1, 1001, s.numel()) + p[s] - p[d]


def _mesh(side):
    v = torch.arange(side * side, device="cuda")
    r, c = v // side, v % side
    s, d = [], []
    for dr, dc in ((0, 1), (0, -1), (1, 0), (-1, 0)):
        ok = (r + dr >= 0) & (r + dr < side) & (c + dc >= 0) & (c + dc < side)
        s.append(v[ok])
        d.append(v[ok] + dr * side + dc)
    return torch.cat(s), torch.cat(d)


def _graph(family, n, deg, seed, mark=False):
    """(offsets, cols, w, src) of a graph; n is the vertex count (er), the
    side of the mesh (grid, road) or the scale (rmat)."""
    g = _gen(seed)
    src = 0
    if family == "er":
        s = _ints(g, 0, n, deg * n)
        d = _ints(g, 0, n - 1, deg * n)
        d = d + (d >= s)
        w = _shifted(g, n, s, d)
        src = int(np.random.default_rng(seed).integers(0, n))
        if mark:
            # three more vertices on a negative cycle that the graph reaches
            t = torch.tensor
            s = torch.cat([s, t([src, n, n + 1, n + 2], device="cuda")])
            d = torch.cat([d, t([n, n + 1, n + 2, n], device="cuda")])
            w = torch.cat([w, t([5, 2, 2, -5], device="cuda")])
            n += 3
    elif family == "rmat":
        scale, n = n, 1 << n
        s = torch.zeros(deg * n, dtype=torch.int64, device="cuda")
        d = torch.zeros_like(s)
        for bit in range(scale):
            q = torch.rand(deg * n, generator=g, device="cuda")
            s |= (q >= 0.76).to(torch.int64) << bit
            d |= (((q >= 0.57) & (q < 0.76)) | (q >= 0.95)).to(torch.int64) << bit
        perm = torch.randperm(n, generator=g, device="cuda")
        s, d = perm[s], perm[d]
        w = _shifted(g, n, s, d)
    elif family == "grid":
        side, n = n, n * n
        s, d = _mesh(side)
        w = _ints(g, 1, 101, s.numel())
    else:
        side, n = n, n * n
        s, d = _mesh(side)
        k = round(0.01 * s.numel())
        r, c = _ints(g, 0, side - 1, k), _ints(g, 0, side - 1, k)
        a, b = r * side + c, (r + 1) * side + c + 1
        flip = torch.rand(k, generator=g, device="cuda") < 0.5
        s, d = torch.cat([s, torch.where(flip, b, a)]), torch.cat([d, torch.where(flip, a, b)])
        w = _shifted(g, n, s, d)
    off, col, w = _csr(n, s, d, w)
    if family == "rmat":
        src = int(torch.argmax(torch.diff(off)))
    return off, col, w, src


_LAUNCH = {
    "default": None,
    "tuned": {"wg_count": 256, "segments": 4, "ticket_batch": 2},
    "buckets": {"bucket_width": 4, "wg_count": 64},
}


def _sizes(case):
    """Vertex counts of a batch's queries (of the case, not of the seed)."""
    rng = np.random.default_rng(case["count"] * 1000003 + case["lo"])
    x = rng.uniform(math.log(case["lo"]), math.log(case["hi"] + 0.5), case["count"])
    return [int(v) for v in np.maximum(np.rint(np.exp(x)), 2)]


def _outputs(sizes, pred=True):
    """One buffer for all queries' distances (and predecessors), and each
    query's part of it."""
    total = sum(sizes)
    dist = torch.empty(total, dtype=torch.int64, device="cuda")
    par = torch.empty(total, dtype=torch.int32, device="cuda") if pred else None
    return dist, par, list(dist.split(sizes)), list(par.split(sizes)) if pred else [None] * len(sizes)


def _batch_graphs(case, seed):
    """[(offsets, cols, w, src)] of a batch's queries."""
    if case["family"] == "rmat":
        off, col, w, _ = _graph("rmat", case["lo"], 16, seed)
        cand = torch.nonzero(torch.diff(off) > 0).flatten().cpu().numpy()
        pick = np.random.default_rng(seed).choice(cand, case["count"], replace=False)
        return [(off, col, w, int(s)) for s in np.sort(pick)]
    return [_graph("er", n, 8, seed * 1000 + i) for i, n in enumerate(_sizes(case))]


def _served_mix(case, seed):
    """Resident graphs, uploaded graphs and the (graph, source) sequence."""
    rng = np.random.default_rng(seed)
    resident = [_graph("rmat", case["scale"], 16, seed), _graph("road", case["side"], 4, seed + 1),
                _graph("er", case["n"], 8, seed + 2)]
    sizes = np.random.default_rng(case["requests"] + case["uploads"])
    up = [_graph("er", int(x), 8, seed + 3 + i) for i, x in
          enumerate(np.exp(sizes.uniform(math.log(2000), math.log(100000), case["uploads"])))]
    seq = []
    for i in range(case["requests"]):
        if up and i % max(1, case["requests"] // len(up)) == 0:
            g = up[i // max(1, case["requests"] // len(up)) % len(up)]
            seq.append((-1, g, g[3]))
        else:
            k = i % 3
            seq.append((k, resident[k], int(rng.integers(0, resident[k][0].numel() - 1))))
    return resident, seq


# ---------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("fifo", "tasks"):
        n = case["items"]
        g = _gen(seed)
        st = {"kind": kind, "queue": bq.Queue(case["capacity"]), "n": n}
        if kind == "fifo":
            st["vals"] = torch.randint(-2**31, 2**31, (n,), generator=g, device="cuda").to(torch.int32)
            st["launch"] = ONE_WAVE
        else:
            st["vals"] = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
            st["result"] = torch.randint(0, 2**31, (n,), generator=g, device="cuda").to(torch.int32)
            st["launch"] = {"ticket_batch": case["b"]} if case["b"] else None
        return st
    if kind == "mixed":
        n = case["ops"] // 2
        return {"kind": kind, "queue": bq.Queue(case["capacity"]), "ops": case["ops"],
                "launch": {"ticket_batch": case["b"]},
                "result": torch.randint(0, 2**31, (n,), generator=_gen(seed), device="cuda").to(torch.int32)}
    if kind in ("sssp", "noalloc", "rounds"):
        off, col, w, src = _graph(case["family"], case["n"], case["deg"], seed,
                                  case.get("mark", False))
        n, m = off.numel() - 1, col.numel()
        st = {"kind": kind, "graph": (off, col, w), "src": src,
              "dist": torch.empty(n, dtype=torch.int64, device="cuda"), "pred": None}
        if case.get("pred", True):
            st["pred"] = torch.empty(n, dtype=torch.int32, device="cuda")
        if kind == "sssp":
            st["ctx"] = bq.SsspContext(n, m)
            st["opts"] = {"launch": _LAUNCH[case["launch"]], "validate": case["validate"],
                          "neg_inf": case["mark"]}
        elif kind == "noalloc":
            st["opts"] = {"launch": _LAUNCH[case["launch"]]}
        else:
            st["ctx"] = bq.RoundsContext(n, m)
            st["opts"] = {"launch": {"ticket_batch": case["b"]} if case["b"] else None}
        return st
    if kind == "batch":
        graphs = _batch_graphs(case, seed)
        sizes = [g[0].numel() - 1 for g in graphs]
        dist, pred, ds, ps = _outputs(sizes, case["pred"])
        return {"kind": kind, "dist": dist, "pred": pred,
                "queries": [(o, c, w, s, d, p) for (o, c, w, s), d, p in zip(graphs, ds, ps)],
                "batch": bq.SsspBatch(len(graphs), sum(sizes), sum(g[1].numel() for g in graphs))}
    resident, seq = _served_mix(case, seed)
    sizes = [g[0].numel() - 1 for _, g, _ in seq]
    dist, pred, ds, ps = _outputs(sizes)
    big = max(sizes), max(g[1].numel() for _, g, _ in seq)
    server = bq.Server(4, 32, 4 * big[0], 4 * big[1], 1 << 28)
    for g in resident:
        server.add_graph(*g[:3])
    host = {}
    reqs = []
    for (k, g, src), d, p in zip(seq, ds, ps):
        r = {"arrival_us": 0.0, "src": src, "dist": d, "pred": p}
        if k >= 0:
            r["graph"] = k
        else:
            if id(g) not in host:
                host[id(g)] = tuple(t.cpu().pin_memory() for t in g[:3])
            r["upload"] = host[id(g)]
        reqs.append(r)
    return {"kind": kind, "server": server, "requests": reqs, "dist": dist, "pred": pred}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    kind = state["kind"]
    if kind == "fifo":
        q = state["queue"]
        ok = q.enqueue(state["vals"], launch=state["launch"])
        return {"enqueued": ok, "out": q.dequeue(state["n"], launch=state["launch"])}
    if kind == "tasks":
        q = state["queue"]
        ok = q.enqueue(state["vals"], launch=state["launch"])
        task = q.dequeue(state["n"], launch=state["launch"]).long()
        out = torch.zeros(state["n"], dtype=torch.int32, device="cuda")
        out.index_add_(0, task, state["result"][task])
        return {"enqueued": ok, "result": out}
    if kind == "mixed":
        st, sent, got = state["queue"].bench_mixed(state["ops"], launch=state["launch"], log=True)
        out = torch.zeros_like(state["result"])
        out.index_add_(0, got, state["result"][sent])
        return {"enq_ok": st["enq_ok"], "deq_ok": st["deq_ok"], "result": out}
    if kind in ("sssp", "rounds"):
        dist, pred, neg = state["ctx"].solve(*state["graph"], state["src"], dist=state["dist"],
                                             pred=state["pred"],
                                             want_pred=state["pred"] is not None, **state["opts"])
        return {"dist": dist, "pred": pred, "neg": neg}
    if kind == "noalloc":
        neg = bq.sssp_bf_noalloc(*state["graph"], state["src"], state["dist"], state["pred"],
                                 **state["opts"])
        return {"dist": state["dist"], "pred": state["pred"], "neg": neg}
    if kind == "batch":
        neg = state["batch"].solve(state["queries"], graph=True)
        return {"dist": state["dist"], "pred": state["pred"], "neg": np.array(neg)}
    resp, _ = state["server"].run(state["requests"])
    return {"dist": state["dist"], "pred": state["pred"],
            "status": np.array([r["status"] for r in resp], dtype=np.int32),
            "reached": np.array([r["reached_edges"] for r in resp], dtype=np.int64)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _nm(family, n, deg, mark=False):
    if family == "er":
        return n + 3 * mark, deg * n + 4 * mark
    if family == "rmat":
        return 1 << n, deg << n
    m = 4 * n * (n - 1)
    return n * n, m + (round(0.01 * m) if family == "road" else 0)


def work(case):
    """Queue: each value read and written once, each result read and written
    once. Queries: the CSR read once, distances and predecessors written
    once, one add and one compare per edge (the least any form needs)."""
    kind = case["kind"]
    if kind == "fifo":
        return {"bytes": 8 * case["items"], "flops": 0}
    if kind == "tasks":
        return {"bytes": 16 * case["items"], "flops": 0}
    if kind == "mixed":
        return {"bytes": 8 * case["ops"], "flops": 0}
    if kind in ("sssp", "noalloc", "rounds"):
        nm = [_nm(case["family"], case["n"], case["deg"], case.get("mark", False))]
    elif kind == "batch":
        if case["family"] == "rmat":
            n, m = _nm("rmat", case["lo"], 16)
            k = case["count"]
            return {"bytes": 8 * (n + 1 + m) + k * 12 * n, "flops": 2 * k * m}
        nm = [(n, 8 * n) for n in _sizes(case)]
    else:
        res = [_nm("rmat", case["scale"], 16), _nm("road", case["side"], 4), (case["n"], 8 * case["n"])]
        nm = [res[i % 3] for i in range(case["requests"])]
    out = 12 if case.get("pred", True) else 8
    return {"bytes": sum(8 * (n + 1) + 8 * m + out * n for n, m in nm),
            "flops": sum(2 * m for _, m in nm)}


# ---------------------------------------------------------------------------
# the outputs from plain tensor operations, in 64-bit integers
# ---------------------------------------------------------------------------
def _reference(graph, src):
    """Distances by rounds over all edges until nothing changes, and the
    smallest tight in-neighbour of each reached vertex."""
    off, col, w = graph
    n = off.numel() - 1
    u = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(off))
    v, w = col.long(), w.long()
    far = 1 << 60
    dist = torch.full((n,), far, dtype=torch.int64, device="cuda")
    dist[src] = 0
    while True:
        before = dist.clone()
        for _ in range(8):
            du = dist[u]
            dist.scatter_reduce_(0, v, torch.where(du < far, du + w, far), "amin")
        if torch.equal(before, dist):
            break
    du = dist[u]
    tight = (du < far) & (du + w == dist[v]) & (v != src)
    pred = torch.full((n,), n, dtype=torch.int64, device="cuda")
    pred.scatter_reduce_(0, v[tight], u[tight], "amin")
    pred = torch.where(pred == n, -1, pred).to(torch.int32)
    reached = int((torch.diff(off) * (dist < far)).sum())
    return torch.where(dist < far, dist, INF), pred, reached


def exact(case, seed):
    kind = case["kind"]
    if kind == "fifo":
        vals = torch.randint(-2**31, 2**31, (case["items"],), generator=_gen(seed), device="cuda")
        return {"enqueued": case["items"], "out": vals.to(torch.int32)}
    if kind == "tasks":
        g = _gen(seed)
        torch.randperm(case["items"], generator=g, device="cuda")
        res = torch.randint(0, 2**31, (case["items"],), generator=g, device="cuda")
        return {"enqueued": case["items"], "result": res.to(torch.int32)}
    if kind == "mixed":
        n = case["ops"] // 2
        res = torch.randint(0, 2**31, (n,), generator=_gen(seed), device="cuda")
        return {"enq_ok": n, "deq_ok": n, "result": res.to(torch.int32)}
    if kind in ("sssp", "noalloc", "rounds"):
        # a marked cycle has no finite rounds; a large mesh takes thousands
        if case.get("mark") or (case["family"] in ("grid", "road") and case["n"] > 700):
            return None
        off, col, w, src = _graph(case["family"], case["n"], case["deg"], seed)
        d, p, _ = _reference((off, col, w), src)
        return {"dist": d, "pred": p if case.get("pred", True) else None, "neg": False}
    if kind == "batch":
        done = [_reference(g[:3], g[3]) for g in _batch_graphs(case, seed)]
        return {"dist": torch.cat([x[0] for x in done]),
                "pred": torch.cat([x[1] for x in done]) if case["pred"] else None,
                "neg": np.zeros(case["count"], dtype=bool)}
    _, seq = _served_mix(case, seed)
    done = [_reference(g[:3], src) for _, g, src in seq]
    return {"dist": torch.cat([x[0] for x in done]), "pred": torch.cat([x[1] for x in done]),
            "status": np.zeros(len(done), dtype=np.int32),
            "reached": np.array([x[2] for x in done], dtype=np.int64)}
