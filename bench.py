"""Benchmark of the hot path on one MI355X.

One step = one pass over the whole path for the measured workload: the
Section IV "Global Mixed" queue run (2^20 int32 slots, 2^26 operations,
even workgroups enqueue, odd workgroups dequeue) followed by one
queue-driven Bellman-Ford solve (init, persistent solver, unpack of
distances and predecessors) on the RMAT scale-20 graph (16.8M edges,
potential-shifted int32 weights) from its highest-degree vertex.

Prints one JSON line. `value` is SSSP GTEPS (reached edges / device time of
the solve, the Graph500 convention); queue Mops/s is reported beside it.
Inputs are resident in HBM before the timed region starts.

    python bench.py [--steps K] [--warmup W] [--no-cpu] [--calib]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import synth  # noqa: E402  (seeded input generators)
from paper_2608_21826_amd.profsum import kernel_source_hash  # noqa: E402  (no GPU work)

HBM_PEAK_GBS = 8000.0           # MI355X HBM3E, published
QUEUE_CAP = 1 << 20
# RMAT-20 solver launch: the workgroup count and ticket batch sssp_autotune
# picks most often on MI355X (256 two-wave workgroups, 128 items per
# dequeue, FIFO order of work), with four queue segments, the best segment
# count at that shape in alternating runs
RMAT20_LAUNCH = {"wg_count": 256, "segments": 4, "ticket_batch": 2}
# Global Mixed queue launch: 256 items per ticket (bulk), 1024-lane
# workgroups, one per CU (the small search below reports its own pick)
QUEUE_LAUNCH = {"ticket_batch": 256, "wg_size": 1024, "wg_count": 256}
QUEUE_OPS = 1 << 26
# algorithmic bytes per unit of work (per dequeued item: row offsets 16 B,
# key RMW 8 B, slot 4 B, ticket read+write 8 B, queue bookkeeping 4 B; per
# scanned edge: col 4 B + weight 4 B + 8 B key atomic; per enqueue: slot 4 B,
# ticket 8 B, key already counted with the edge, 4 B bookkeeping: Alg. 1's
# queue; the sweep form's items have no tickets)
BYTES_PER_DEQ = 40
BYTES_PER_EDGE = 16
BYTES_PER_PUSH = 16
PMC_FILE = os.path.join(ROOT, "profiles", "sssp_rmat20_pmc.txt")


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


TCC_FILE = os.path.join(ROOT, "profiles", "sssp_rmat20_tcc.txt")
QUEUE_PMC_FILE = os.path.join(ROOT, "profiles", "queue_mixed_b256.txt")


def read_counter_summary(path, kernel, key):
    """One value of a kernel's block in a committed counter summary, or None
    when the file is missing or was taken on other solver sources."""
    if not os.path.exists(path):
        return None
    cur, rec = None, {}
    for line in open(path):
        if line.startswith("#") or "=" not in line:
            continue
        k, v = (x.strip() for x in line.split("=", 1))
        if k == "kernel":
            cur = v
        elif cur == kernel:
            rec[k] = v
    if rec.get("kernel_source_hash") != kernel_source_hash(kernel) or key not in rec:
        return None
    try:
        return float(rec[key])
    except ValueError:
        return None


def cpu_baseline(g, m_reached, budget_s=12.0):
    """The oracle as it stands (round-based Bellman-Ford, Alg. 3 on one
    processing element, single thread) on the same graph and source, repeated
    until about budget_s of CPU time."""
    import oracle
    oracle.load()
    times = []
    t_all = time.perf_counter()
    while True:
        t0 = time.perf_counter()
        _, neg, rounds = oracle.bf_rounds(g)
        times.append(time.perf_counter() - t0)
        if time.perf_counter() - t_all > budget_s or len(times) >= 30:
            break
    t = float(np.mean(times))
    return {"value": m_reached / t / 1e9, "unit": "GTEPS", "cores": 1, "kind": "oracle",
            "sample": f"{len(times)} full solves of the measured RMAT-20 query with the "
                      f"round-based oracle ({rounds} rounds each, mean {t * 1e3:.0f} ms); the "
                      f"queue leg is not timed on the CPU"}


def cpu_baselines_more(g, m_reached, budget_s=5.0):
    """Beside the oracle: the sequential FIFO form (the method's own
    single-thread form, 1 core) and the same rounds as Jacobi rounds on all
    host cores (OpenMP, threads as the environment allows). The transposed
    graph for the latter is built outside the timed loop."""
    import oracle
    out = {}
    times = []
    t_all = time.perf_counter()
    while time.perf_counter() - t_all < budget_s and len(times) < 20:
        t0 = time.perf_counter()
        _, neg, pops, relax = oracle.bf_fifo(g)
        times.append(time.perf_counter() - t0)
    t = float(np.mean(times))
    out["fifo_1core"] = {"value": round(m_reached / t / 1e9, 4), "unit": "GTEPS", "cores": 1,
                         "kind": "oracle_fifo",
                         "sample": f"{len(times)} solves, mean {t * 1e3:.0f} ms, "
                                   f"k = {relax / m_reached:.2f}"}
    csc = oracle.transpose(g)
    times = []
    t_all = time.perf_counter()
    while time.perf_counter() - t_all < budget_s and len(times) < 20:
        t0 = time.perf_counter()
        _, neg, rounds, threads = oracle.bf_jacobi(g, csc)
        times.append(time.perf_counter() - t0)
    t = float(np.mean(times))
    out["jacobi_all_cores"] = {"value": round(m_reached / t / 1e9, 4), "unit": "GTEPS",
                               "cores": threads, "kind": "parallel_rounds",
                               "sample": f"{len(times)} solves, {rounds} Jacobi rounds each, "
                                         f"mean {t * 1e3:.0f} ms"}
    return out


def queue_roofline(ms, launch, b1_ms, probes):
    """Roofline of the Global Mixed queue run (k_bench_mixed).

    Bulk (the timed launch, 64*b items per ticket): 12 algorithmic bytes
    per operation (4 B payload, 4 B ticket read, 4 B ticket write) against
    HBM. One ticket per wave (b = 1): the broker count word takes one
    contended atomic per wave operation, 2^26 / 64 of them at least, and a
    single word serializes its atomics; the peak is the measured rate of
    one contended word (probe of leader-lane atomicAdds)."""
    b = int(launch.get("ticket_batch", 1))
    bulk = QUEUE_OPS * 12 / (ms * 1e-3) / 1e9
    traffic = None
    if launch == QUEUE_LAUNCH:  # the committed counters were taken at this launch
        traffic = read_counter_summary(QUEUE_PMC_FILE, "k_bench_mixed", "hbm_bytes_per_launch")
    res = {"bulk": {"bound": "hbm", "achieved": round(bulk, 1), "peak": HBM_PEAK_GBS,
                    "unit": "GB/s", "frac": round(bulk / HBM_PEAK_GBS, 4),
                    "traffic": traffic, "algorithmic_bytes": QUEUE_OPS * 12, "ticket_batch": b,
                    "kernel": "k_bench_mixed", "kernel_ms": round(ms, 4)}}
    word = None
    if probes:
        word = probes.get("atomic_add_one_word_leader_Mops_w4096")
    if b1_ms:
        atom = (QUEUE_OPS // 64) / (b1_ms * 1e-3) / 1e6
        res["one_ticket_per_wave"] = {
            "bound": "contended_atomic", "achieved": round(atom, 1),
            "peak": word, "unit": "M atomics/s on the count word",
            "frac": round(atom / word, 4) if word else None,
            "atomics_on_count_word": QUEUE_OPS // 64, "kernel_ms": round(b1_ms, 3)}
    return res


def cpu_graph_baselines(graphs, budget_s=4.0):
    """The oracle beside the grid and road legs: its rounds (Alg. 3 on one
    processing element, 1 core), the sequential FIFO form (1 core) and the
    Jacobi rounds on all host cores, each repeated for about budget_s (at
    least once). `graphs`: (label, graph, which of the three to run)."""
    import oracle
    out = {}

    def timed(fn):
        times = []
        t_all = time.perf_counter()
        while True:
            t0 = time.perf_counter()
            r = fn()
            times.append(time.perf_counter() - t0)
            if time.perf_counter() - t_all > budget_s or len(times) >= 20:
                return float(np.median(times)), len(times), r

    for label, g, kinds in graphs:
        d = {}
        if "rounds" in kinds:
            t, k, (dist, neg, rounds) = timed(lambda: oracle.bf_rounds(g))
            mr = int(np.diff(g.offsets)[dist != oracle.INF].sum())
            d["oracle_rounds_1core"] = {"value": round(mr / t / 1e9, 5), "unit": "GTEPS",
                                        "cores": 1, "kind": "oracle", "ms": round(t * 1e3, 2),
                                        "sample": f"{k} full solves, {rounds} rounds each"}
        if "fifo" in kinds:
            t, k, (dist, neg, pops, rel) = timed(lambda: oracle.bf_fifo(g))
            mr = int(np.diff(g.offsets)[dist != oracle.INF].sum())
            d["fifo_1core"] = {"value": round(mr / t / 1e9, 5), "unit": "GTEPS", "cores": 1,
                               "kind": "oracle_fifo", "ms": round(t * 1e3, 2),
                               "sample": f"{k} full solves, k = {rel / max(mr, 1):.1f}"}
        if "jacobi" in kinds:
            csc = oracle.transpose(g)
            t, k, (dist, neg, rounds, threads) = timed(lambda: oracle.bf_jacobi(g, csc))
            mr = int(np.diff(g.offsets)[dist != oracle.INF].sum())
            d["jacobi_all_cores"] = {"value": round(mr / t / 1e9, 5), "unit": "GTEPS",
                                     "cores": threads, "kind": "parallel_rounds",
                                     "ms": round(t * 1e3, 2),
                                     "sample": f"{k} full solves, {rounds} Jacobi rounds each"}
        out[label] = d
        log(f"cpu {label}: {d}")
    return out


def host_info():
    model = None
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return {"cpu_model": model, "nproc": os.cpu_count(),
            "omp_num_threads": os.environ.get("OMP_NUM_THREADS")}


def cpu_queue_baselines(threads=None):
    """The queue on the host (bounded samples): a sequential ring on one core
    running the Global Mixed sequence (2^26 operations), and Alg. 1's Broker
    Queue with C11 atomics on all host threads (2^22 operations, 2^20 slots)."""
    import oracle
    threads = threads or max(2, (os.cpu_count() or 2))
    threads = int(os.environ.get("OMP_NUM_THREADS", threads))
    t_ring = min(oracle.ring_mixed(QUEUE_CAP, QUEUE_OPS) for _ in range(2))
    n = 1 << 22
    t_bq, fails, _, _ = oracle.bq_mixed(QUEUE_CAP, n, threads)
    return {"ring_1core": {"value": round(QUEUE_OPS / t_ring / 1e6, 1), "unit": "Mops/s",
                           "cores": 1, "kind": "sequential_ring",
                           "sample": "2^26 operations alternating enqueue / dequeue"},
            "bq_model_all_threads": {"value": round(n / t_bq / 1e6, 2), "unit": "Mops/s",
                                     "cores": threads, "kind": "broker_queue_cpu_model",
                                     "sample": f"2^22 operations (Global Mixed), 2^20 slots, "
                                               f"{fails} Full/Empty retries"}}


def run_probes(pkg, torch, dev):
    """Measured peaks of the resources the solver uses (context for the
    roofline; the reported peak stays the published HBM figure)."""
    cus = pkg.device_cus()
    res = {"cus": cus}
    nbytes = 1 << 30
    a = torch.empty(nbytes // 8, dtype=torch.int64, device=dev)
    b = torch.empty_like(a)
    pkg.probe(0, a, b, size=nbytes, grid=8 * cus, block=256)
    ms = min(pkg.probe(0, a, b, size=nbytes, grid=8 * cus, block=256) for _ in range(5))
    res["hbm_copy_GBs"] = round(2 * nbytes / ms / 1e6, 1)
    del a, b
    sink = torch.zeros(2, dtype=torch.int64, device=dev)
    for words, name in ((1 << 20, "8MiB"), (1 << 25, "256MiB")):
        t = torch.full((words,), 2**62, dtype=torch.int64, device=dev)
        grid, block, opl = 8 * cus, 256, 64
        pkg.probe(1, t, sink, size=words, ops_per_lane=opl, grid=grid, block=block)
        ms = min(pkg.probe(1, t, sink, size=words, ops_per_lane=opl, grid=grid, block=block)
                 for _ in range(3))
        res[f"atomic_min_rand_{name}_Gops"] = round(grid * block * opl / ms / 1e6, 2)
        pkg.probe(5, t, sink, size=words, ops_per_lane=opl, grid=grid, block=block)
        ms = min(pkg.probe(5, t, sink, size=words, ops_per_lane=opl, grid=grid, block=block)
                 for _ in range(3))
        res[f"load_rand_{name}_Gops"] = round(grid * block * opl / ms / 1e6, 2)
        del t
    word = torch.zeros(2, dtype=torch.int64, device=dev)
    grid, block, opl = 4 * cus, 256, 8
    pkg.probe(2, word, None, ops_per_lane=opl, grid=grid, block=block)
    ms = min(pkg.probe(2, word, None, ops_per_lane=opl, grid=grid, block=block) for _ in range(3))
    res["atomic_add_one_word_Mops"] = round(grid * block * opl / ms / 1e3, 1)
    for kind, name in ((3, "atomic_add_one_word_leader_Mops"), (4, "load_one_word_leader_Mops")):
        for grid in (256, 1024, 4096):
            opl = 64
            pkg.probe(kind, word, None, ops_per_lane=opl, grid=grid, block=256)
            ms = min(pkg.probe(kind, word, None, ops_per_lane=opl, grid=grid, block=256)
                     for _ in range(3))
            res[f"{name}_w{grid * 4}"] = round(grid * 4 * opl / ms / 1e3, 1)
    return res


def reached_edges(torch, dist, deg_t):
    return int(deg_t[dist != np.iinfo(np.int64).max].sum().item())


GOLDEN_DIR = os.path.join(ROOT, "tests", "golden")


def golden(name):
    """Stored result of a full-size configuration (written by
    tests/golden/make_golden.py from the CPU oracle and certified there by
    an independent algorithm)."""
    fname = {"grid64": "grid64.json", "rmat20": "rmat20.json",
             "rmat20_x64_sources": "rmat20.json", "road2048": "road2048.json",
             "road2048_negcycle": "road2048.json", "er256": "er256.json"}[name]
    with open(os.path.join(GOLDEN_DIR, fname)) as f:
        return json.load(f)[name]


def sha256(a) -> str:
    import hashlib
    return hashlib.sha256(np.ascontiguousarray(a).tobytes()).hexdigest()


def graph_sha256(g) -> str:
    import hashlib
    h = hashlib.sha256()
    for a in (g.offsets, g.cols, g.w):
        h.update(np.ascontiguousarray(a).tobytes())
    return h.hexdigest()


def matches_golden(rec, dist, pred) -> bool:
    """dist / pred (device tensors) equal the stored result byte for byte."""
    return (sha256(dist.cpu().numpy()) == rec["dist_sha256"] and
            sha256(pred.cpu().numpy()) == rec["pred_sha256"])


def road_tune(pkg, torch, dev, g):
    """The library autotuner on the road mesh (it picks near / far buckets
    there): returns its launch, as a dict of the fields it set."""
    off = torch.from_numpy(g.offsets).to(dev)
    col = torch.from_numpy(g.cols).to(dev)
    w = torch.from_numpy(g.w).to(dev)
    ctx = pkg.SsspContext(g.n, g.m)
    try:
        L, ms = ctx.autotune(off, col, w, g.src, reps=3)
    finally:
        ctx.close()
    log(f"road2048 autotune: {L} {ms:.2f} ms")
    return {k: v for k, v in L.items() if v}


def graph_leg(pkg, torch, dev, name, g, reps, warmup, launch=None, ctx=None):
    """Solves of one configuration at a fixed launch (the library default
    unless given): median device time over `reps` HIP-event-timed solves
    after `warmup` untimed ones; reached-edge GTEPS; work ratio; every
    solve's output checked against the stored result (outside the timing)."""
    rec = golden(name)
    assert graph_sha256(g) == rec["graph_sha256"], f"{name}: generator output changed"
    off = torch.from_numpy(g.offsets).to(dev)
    col = torch.from_numpy(g.cols).to(dev)
    w = torch.from_numpy(g.w).to(dev)
    own = ctx is None
    if own:
        ctx = pkg.SsspContext(g.n, g.m)
    dist = torch.empty(g.n, dtype=torch.int64, device=dev)
    pred = torch.empty(g.n, dtype=torch.int32, device=dev)
    try:
        for _ in range(warmup):
            ctx.solve(off, col, w, g.src, dist=dist, pred=pred, launch=launch)
        ms, kms, rel, exact = [], [], [], True
        for _ in range(reps):
            _, _, neg = ctx.solve(off, col, w, g.src, dist=dist, pred=pred, launch=launch)
            st = ctx.stats()
            ms.append(st["ms"])
            kms.append(st["solve_ms"])
            rel.append(st["relaxations"])
            exact &= (not neg) and matches_golden(rec, dist, pred)
        grid = int(st["grid"])
    finally:
        if own:
            ctx.close()
    med = float(np.median(ms))
    mr = rec["m_reached"]
    return {"ms_median": round(med, 4), "ms_min": round(float(np.min(ms)), 4),
            "solver_kernel_ms": round(float(np.median(kms)), 4),
            "gteps": round(mr / (med * 1e-3) / 1e9, 4), "m_reached": mr,
            "work_ratio_k": round(float(np.mean(rel)) / mr, 3), "grid": grid,
            "launch": launch or "library default", "runs": reps,
            "parity": "exact" if exact else "MISMATCH"}


def negcycle_leg(pkg, torch, dev, g, reps=3, launch=None):
    """Detection of the planted negative 3-cycle: device time of the solve
    until the flag is final (HIP events around init, solve and unpack)."""
    rec = golden("road2048_negcycle")
    assert graph_sha256(g) == rec["graph_sha256"], "road2048_negcycle: generator output changed"
    off = torch.from_numpy(g.offsets).to(dev)
    col = torch.from_numpy(g.cols).to(dev)
    w = torch.from_numpy(g.w).to(dev)
    ctx = pkg.SsspContext(g.n, g.m)
    try:
        ms, flags, walks = [], [], []
        for _ in range(reps):
            _, _, neg = ctx.solve(off, col, w, g.src, launch=launch)
            st = ctx.stats()
            ms.append(st["ms"])
            flags.append(bool(neg))
            walks.append(st["walks"])
    finally:
        ctx.close()
    return {"detect_ms_median": round(float(np.median(ms)), 3),
            "detect_ms_max": round(float(np.max(ms)), 3), "runs": reps,
            "flag": int(all(flags)), "parity": "exact" if all(flags) == rec["neg_cycle"]
            else "MISMATCH", "parent_walks": int(np.median(walks))}


def batched_leg(pkg, torch, dev, name, queries, graphs, steps, single_launch=None,
                batch_launch=None, check=None):
    """One batched launch over all queries vs the same queries one sssp_bf
    call at a time (each a separate synchronous call). Device time from HIP
    events in both cases; reached edges summed over the queries. The batched
    launch is autotuned unless batch_launch fixes it."""
    tn = sum(g.n for g in graphs)
    tm = sum(g.m for g in graphs)
    b = pkg.SsspBatch(len(queries), tn, tm)
    if batch_launch is None:
        launch, tune_ms = b.autotune(queries)
        log(f"{name}: batch autotune {launch} {tune_ms:.3f} ms")
    else:
        launch = dict(batch_launch)
    for _ in range(2):
        b.solve(queries, launch=launch, graph=True)
    ms = []
    for _ in range(steps):
        b.solve(queries, launch=launch, graph=True)
        ms.append(b.stats()["ms"])
    st = b.stats()
    # the batched outputs (before the one-at-a-time solves overwrite them)
    parity = check(queries) if check is not None else None
    degs = {}
    m_reached = 0
    for (off, col, w, src, dist, pred), g in zip(queries, graphs):
        key = id(g)
        if key not in degs:
            degs[key] = torch.diff(off)
        m_reached += reached_edges(torch, dist, degs[key])
    b.close()
    # one query at a time
    mx = max(g.n for g in graphs)
    mm = max(g.m for g in graphs)
    ctx = pkg.SsspContext(mx, mm)
    for q in queries[:2]:
        ctx.solve(q[0], q[1], q[2], q[3], dist=q[4], pred=q[5], launch=single_launch)
    one_ms = []
    t0 = time.perf_counter()
    for q in queries:
        ctx.solve(q[0], q[1], q[2], q[3], dist=q[4], pred=q[5], launch=single_launch)
        one_ms.append(ctx.stats()["ms"])
    one_wall = (time.perf_counter() - t0) * 1e3
    ctx.close()
    bms = float(np.median(ms))
    return {"queries": len(queries), "m_reached": m_reached,
            "batched_ms": round(bms, 3), "batched_gteps": round(m_reached / bms / 1e6, 3),
            "one_at_a_time_ms": round(float(np.sum(one_ms)), 3),
            "one_at_a_time_wall_ms": round(one_wall, 3),
            "one_at_a_time_gteps": round(m_reached / float(np.sum(one_ms)) / 1e6, 3),
            "speedup": round(float(np.sum(one_ms)) / bms, 2),
            "launch": launch, "relaxations": int(st["relaxations"]),
            **({"parity": parity} if parity is not None else {})}


def certify_sssp(torch, off, col, w, src, dist, pred) -> bool:
    """A shortest-path certificate, checked with tensor ops on the GPU (no
    oracle): d[src] = 0; no edge from a reached vertex can lower its target
    (d[v] <= d[u] + w); pred[v] is the smallest u with d[u] + w = d[v], -1 for
    the source and for unreached vertices; every reached vertex other than the
    source has such a u. On graphs whose cycles all weigh more than zero (the
    potential-shifted graphs here: every cycle weighs its w0 >= 1 per edge)
    the tight edges form no cycle, so following pred from any reached vertex
    ends at the source along a path of weight d[v]; with the edge condition
    that makes d the exact distances."""
    inf = torch.iinfo(torch.int64).max
    n = off.numel() - 1
    tails = torch.repeat_interleave(torch.arange(n, device=off.device), torch.diff(off))
    du = dist[tails]
    fin = du != inf
    cand = du[fin] + w[fin].to(torch.int64)
    heads = col[fin].to(torch.int64)
    if int(dist[src].item()) != 0 or not bool((dist[heads] <= cand).all().item()):
        return False
    tight = dist[heads] == cand
    best = torch.full((n,), n, dtype=torch.int64, device=off.device)
    best.scatter_reduce_(0, heads[tight], tails[fin][tight], reduce="amin")
    want = torch.where(best == n, torch.full_like(best, -1), best)
    want[src] = -1
    reached = dist != inf
    want[~reached] = -1
    if int((want[reached] >= 0).sum().item()) != int(reached.sum().item()) - 1:
        return False
    return bool(torch.equal(pred.to(torch.int64), want))


def served_leg(pkg, torch, dev, g_rmat, t_rmat, n_req, seed=0, lanes=4, road_launch=None,
               pool=20, calib=200, check_n=200):
    """Served form (Poisson arrivals over 3 resident graphs + one-off ER
    uploads): the continuous-batching engine vs the same engine limited to
    one query per launch and one lane (sequential one-query launches), at
    1.5x and 0.5x the sequential service rate, n_req requests each. 90 % of
    the requests hit the resident graphs (RMAT-20, road2048, ER-200k), 10 %
    upload an ER graph drawn from a pool of `pool` graphs with n log-uniform
    in [1e4, 2e6]. The sequential service rate comes from a closed-loop run
    of the first `calib` requests of the mix on the sequential engine.
    Large road2048 requests run with `road_launch` (near / far buckets).
    p50/p99 latency from arrival to completion; GTEPS = reached edges of all
    requests / wall time. After the timed runs, the first `check_n` requests
    of the mix run again on the continuous-batching engine into caller
    buffers, and every answer is checked with `certify_sssp`."""
    rng = np.random.default_rng(synth.SEED_BASE + 4 + seed)
    road = synth.config_graph("road2048")
    er = synth.config_graph("er200k")
    resident = [g_rmat, road, er]
    dev_csr = [t_rmat] + [(torch.from_numpy(x.offsets).to(dev), torch.from_numpy(x.cols).to(dev),
                           torch.from_numpy(x.w).to(dev)) for x in (road, er)]
    up_sizes = np.rint(np.exp(rng.uniform(np.log(1e4), np.log(2e6), size=pool))).astype(int)
    t0 = time.time()
    uploads = [synth.erdos_renyi(int(nv), 8, seed=synth.SEED_BASE + 40 + i)
               for i, nv in enumerate(up_sizes)]
    pinned = [(torch.from_numpy(x.offsets).pin_memory(), torch.from_numpy(x.cols).pin_memory(),
               torch.from_numpy(x.w).pin_memory()) for x in uploads]
    log(f"served: {pool} upload graphs ({int(up_sizes.sum())} vertices) in "
        f"{time.time() - t0:.1f}s")
    srcs = [synth.random_sources(x, n_req, seed=synth.SEED_BASE + 50 + i)
            for i, x in enumerate(resident)]
    mix = []
    for i in range(n_req):
        if rng.random() < 0.1:
            k = int(rng.integers(0, len(uploads)))
            mix.append(("u", k, int(rng.integers(0, uploads[k].n))))
        else:
            k = int(rng.integers(0, 3))
            mix.append(("g", k, int(srcs[k][i % len(srcs[k])])))
    max_n = 8 * max(x.n for x in resident + uploads)
    max_m = 8 * max(x.m for x in resident + uploads)

    def trace(arrivals, count):
        out = []
        for t, (kind, k, src) in zip(arrivals, mix[:count]):
            r = {"arrival_us": float(t), "src": src}
            if kind == "u":
                r["upload"] = pinned[k]
            else:
                r["graph"] = k
            out.append(r)
        return out

    def run(lanes, max_batch, arrivals):
        srv = pkg.Server(lanes, max_batch, max_n, max_m, 4 << 30)
        try:
            for c in dev_csr:
                srv.add_graph(*c)
            if road_launch:
                srv.set_graph_launch(1, road_launch)
            srv.run(trace(np.zeros(4), 4))  # warm-up
            resp, st = srv.run(trace(arrivals, len(arrivals)))
        finally:
            srv.close()
        lat = np.array([x["latency_us"] for x in resp]) / 1e3
        bad = sum(1 for x in resp if x["status"] != 0)
        edges = sum(x["reached_edges"] for x in resp)
        return {"requests": len(resp), "p50_ms": round(float(np.percentile(lat, 50)), 3),
                "p99_ms": round(float(np.percentile(lat, 99)), 3),
                "mean_ms": round(float(lat.mean()), 3), "wall_ms": round(st["wall_ms"], 1),
                "gteps": round(edges / (st["wall_ms"] * 1e6), 3), "launches": st["launches"],
                "max_lanes_busy": st["max_lanes_busy"], "max_inflight": st["max_inflight"],
                "failed": bad}

    # sequential service time (closed loop: the first `calib` requests queued at t=0)
    seq0 = run(1, 1, np.zeros(min(calib, n_req)))
    mean_service_ms = seq0["wall_ms"] / seq0["requests"]
    res = {"requests": n_req, "upload_pool": pool, "calibration_requests": seq0["requests"],
           "mean_sequential_service_ms": round(mean_service_ms, 3),
           "road2048_launch": road_launch}
    for load in (1.5, 0.5):
        qps = load * 1e3 / mean_service_ms
        arr = np.cumsum(rng.exponential(1e6 / qps, size=n_req))
        res[f"qps_{load}x"] = {"qps": round(qps, 2),
                               "continuous_batching": run(lanes, 32, arr),
                               "sequential": run(1, 1, arr)}
        log(f"served {load}x: {res[f'qps_{load}x']}")
    # the engine's answers: the head of the mix again, at 1.5x the
    # sequential rate, into caller buffers, each certified on the GPU
    count = min(check_n, n_req)
    reqs = trace(np.cumsum(rng.exponential(mean_service_ms * 1e3 / 1.5, size=count)), count)
    csr_of = []
    for r, (kind, k, src) in zip(reqs, mix[:count]):
        x = uploads[k] if kind == "u" else resident[k]
        r["dist"] = torch.empty(x.n, dtype=torch.int64, device=dev)
        r["pred"] = torch.empty(x.n, dtype=torch.int32, device=dev)
        csr_of.append(("u", k) if kind == "u" else ("g", k))
    srv = pkg.Server(lanes, 32, max_n, max_m, 4 << 30)
    try:
        for c in dev_csr:
            srv.add_graph(*c)
        if road_launch:
            srv.set_graph_launch(1, road_launch)
        resp, _ = srv.run(reqs)
    finally:
        srv.close()
    up_dev = {}
    ok = all(x["status"] == 0 and x["neg_cycle"] == 0 for x in resp)
    for r, (kind, k) in zip(reqs, csr_of):
        if not ok:
            break
        if kind == "g":
            off_, col_, w_ = dev_csr[k]
        else:
            if k not in up_dev:
                up_dev[k] = tuple(torch.from_numpy(a).to(dev) for a in
                                  (uploads[k].offsets, uploads[k].cols, uploads[k].w))
            off_, col_, w_ = up_dev[k]
        ok = certify_sssp(torch, off_, col_, w_, r["src"], r["dist"], r["pred"])
    res["parity"] = f"exact (first {count} requests, certified)" if ok else "MISMATCH"
    log(f"served parity: {res['parity']}")
    return res


def queue_sweep(pkg, steps=2):
    """The paper's Section IV queue sweep, on wave64 hardware: both scenarios
    (Global Mixed, Global EnqDeq), both policies (Broker Queue, BWD),
    workgroup sizes 64..1024 (the paper's 32..512 threads per block, in whole
    waves), workgroup counts from the paper's 64/108/216 blocks up to the
    co-resident grid, and ticket batch b = 1 (one wave op per 64 lanes) and 16;
    plus the partitioned queue (8 segments, one per XCD) under the Broker
    Queue policy. Mixed: 2^20 slots, 2^26 operations. EnqDeq: 2^26 operations on a queue
    of 2^25 slots, so that every one of the 2^25 enqueues fits and each
    phase moves real items. Returns rows of Mops/s."""
    qm = pkg.Queue(QUEUE_CAP)
    qe = pkg.Queue(QUEUE_OPS // 2)
    rows = []
    for scen in ("mixed", "enqdeq"):
        q = qm if scen == "mixed" else qe
        for bwd, seg in ((False, 1), (True, 1), (False, 8)):
            for b in (1, 16):
                for wgsz in (64, 128, 256, 512, 1024):
                    for wgs in (64, 108, 216, 512, 0):
                        if seg > 1 and wgs in (108, 216):
                            continue  # not a multiple of 2 x 8 workgroups
                        L = {"ticket_batch": b, "wg_size": wgsz, "wg_count": wgs,
                             "flags": pkg.BQ_F_BWD if bwd else 0, "segments": seg}
                        best = None
                        for _ in range(steps):
                            if scen == "mixed":
                                st = q.bench_mixed(QUEUE_OPS, launch=L)[0]
                                ms, fails = st["ms"], st["enq_full"] + st["deq_empty"]
                                ok = st["enq_ok"] + st["deq_ok"]
                            else:
                                e, d = q.bench_enqdeq(QUEUE_OPS, launch=L)
                                ms, fails = e["ms"] + d["ms"], e["enq_full"] + d["deq_empty"]
                                ok = e["enq_ok"] + d["deq_ok"]
                            if best is None or ms < best[0]:
                                best = (ms, fails, ok)
                        rows.append({"scenario": scen, "policy": "BWD" if bwd else "BQ", "b": b,
                                     "segments": seg,
                                     "wg_size": wgsz, "wg_count": wgs, "ms": round(best[0], 3),
                                     "mops": round(QUEUE_OPS / best[0] / 1e3, 1),
                                     "refused": int(best[1]), "ok": int(best[2])})
    qm.close()
    qe.close()
    return rows


def rounds_leg(pkg, torch, g, off, col, w, ref_dist, m_reached, reps=5):
    """The paper's own form on the same graph: round-based Bellman-Ford with
    the queue holding edges (every round relaxes all m edges). Ticket batch
    b = 4, 16, 64 tried; the distances must equal the queue solver's."""
    rc = pkg.RoundsContext(g.n, g.m)
    best = None
    for b in (4, 16, 64):
        L = {"ticket_batch": b}
        for _ in range(reps):
            d, _, neg = rc.solve(off, col, w, g.src, launch=L, want_pred=True)
            assert not neg and torch.equal(d, ref_dist), "rounds form: distances differ"
            st = rc.stats()
            if best is None or st["ms"] < best[0]["ms"]:
                best = (st, b)
    rc.close()
    st, b = best
    return {"ms": round(st["ms"], 3), "gteps": round(m_reached / (st["ms"] * 1e-3) / 1e9, 4),
            "rounds": int(st["rounds"]), "relaxations": int(st["relaxations"]),
            "changes": int(st["changes"]), "ticket_batch": b, "grid": int(st["grid"]),
            "relax_per_s_G": round(st["relaxations"] / (st["solve_ms"] * 1e-3) / 1e9, 3)}


def bf_sweep(pkg, torch, dev, steps=3):
    """Queue-driven Bellman-Ford under both broker policies (Broker Queue,
    BWD), with one queue and with 2 and 8 segments, over the paper's block
    counts 64 / 108 / 216, then 512 and the co-resident maximum (8 per CU is
    more than fits; the library clamps), for ticket batch b = 1 and 4, at the
    default row chunk, on RMAT-20 and the 2048^2 road graph. Every run's
    distances must equal the first run's. Returns rows of GTEPS."""
    rows = []
    for name in ("rmat20", "road2048"):
        g = synth.config_graph(name)
        off = torch.from_numpy(g.offsets).to(dev)
        col = torch.from_numpy(g.cols).to(dev)
        w = torch.from_numpy(g.w).to(dev)
        ctx = pkg.SsspContext(g.n, g.m)
        ref, _, neg = ctx.solve(off, col, w, g.src, validate=True)
        assert not neg
        ref = ref.clone()
        reached = (ref != np.iinfo(np.int64).max).cpu().numpy()
        m_reached = int(np.diff(g.offsets)[reached].sum())
        for bwd, seg in ((False, 1), (True, 1), (False, 2), (True, 2), (False, 8), (True, 8)):
            for b in (1, 4):
                for wgs in (64, 108, 216, 512, 8 * pkg.device_cus()):
                    L = {"ticket_batch": b, "wg_count": wgs,
                         "flags": pkg.BQ_F_BWD if bwd else 0, "segments": seg}
                    best = None
                    for _ in range(steps):
                        d, _, neg = ctx.solve(off, col, w, g.src, launch=L)
                        assert not neg and torch.equal(d, ref), f"{name} {L}: distances differ"
                        st = ctx.stats()
                        if best is None or st["ms"] < best["ms"]:
                            best = st
                    rows.append({"graph": name, "policy": "BWD" if bwd else "BQ", "b": b,
                                 "segments": seg,
                                 "wg_count": int(best["grid"]), "ms": round(best["ms"], 3),
                                 "gteps": round(m_reached / (best["ms"] * 1e-3) / 1e9, 3),
                                 "k": round(best["relaxations"] / m_reached, 3),
                                 "idle_polls": int(best["idle_polls"])})
                    log(f"bf sweep {rows[-1]}")
        ctx.close()
        del off, col, w, ref
    return rows


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle baselines")
    ap.add_argument("--calib", action="store_true",
                    help="also run a 1 GiB copy kernel (byte-counter calibration)")
    ap.add_argument("--scale", type=int, default=20)
    ap.add_argument("--sssp-launch", type=str, default=None,
                    help='fixed solver launch as JSON, e.g. {"wg_count":128,"row_chunk":256}')
    ap.add_argument("--queue-launch", type=str, default=None,
                    help='fixed queue launch as JSON, e.g. {"ticket_batch":64,"wg_size":1024}')
    ap.add_argument("--no-tune", action="store_true",
                    help="library default launch shapes (no autotuning)")
    ap.add_argument("--tune", action="store_true",
                    help="time the RMAT-20 solve and the queue at this run's autotuner / "
                         "search picks instead of the fixed launches")
    ap.add_argument("--sssp-only", action="store_true",
                    help="skip every leg but the timed RMAT-20 solves (counter passes)")
    ap.add_argument("--queue-only", action="store_true",
                    help="only the timed queue runs (counter passes on k_bench_mixed)")
    ap.add_argument("--no-batched", action="store_true",
                    help="skip the batched-vs-one-at-a-time legs")
    ap.add_argument("--no-graphs", action="store_true",
                    help="skip the grid and road legs")
    ap.add_argument("--served-requests", type=int, default=2000,
                    help="requests per served run (0 skips the served leg)")
    ap.add_argument("--served-lanes", type=int, default=4,
                    help="lanes of the continuous-batching engine in the served leg")
    ap.add_argument("--queue-sweep", action="store_true",
                    help="only run the queue scenario / policy / launch-shape sweep")
    ap.add_argument("--bf-sweep", action="store_true",
                    help="only run the solver policy / workgroup-count sweep")
    ap.add_argument("--no-probes", action="store_true",
                    help="skip the HBM copy and atomic-rate probes (roofline context)")
    ap.add_argument("--batched-launch", type=str, default=None,
                    help='fixed launch of the batched legs as JSON (no autotuning), '
                         'e.g. {"wg_count":512,"ticket_batch":1}')
    ap.add_argument("--batched-only", choices=("rmat20x64", "er256"), default=None,
                    help="run only this batched workload (for counter passes)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}); the multi-GPU form of "
              "this path is not built.", file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2608_21826_amd as pkg

    if args.queue_sweep:
        for row in queue_sweep(pkg):
            print(json.dumps(row), flush=True)
        return

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.bf_sweep:
        for row in bf_sweep(pkg, torch, dev):
            print(json.dumps(row), flush=True)
        return
    only_timed = args.sssp_only or args.queue_only

    t0 = time.time()
    g = synth.rmat(args.scale)
    log(f"graph rmat{args.scale}: n={g.n} m={g.m} src={g.src} ({time.time() - t0:.1f}s)")
    rec = golden("rmat20") if args.scale == 20 else None
    if rec is not None:
        assert graph_sha256(g) == rec["graph_sha256"], "rmat20: generator output changed"
    off = torch.from_numpy(g.offsets).to(dev)
    col = torch.from_numpy(g.cols).to(dev)
    w = torch.from_numpy(g.w).to(dev)
    ctx = pkg.SsspContext(g.n, g.m)
    q = pkg.Queue(QUEUE_CAP)
    # every library object is closed explicitly, before the interpreter and
    # the HIP runtime shut down
    try:
        out, parity_ok = run_main_legs(args, pkg, torch, dev, g, rec, off, col, w, ctx, q,
                                       only_timed)
    finally:
        ctx.close()
        q.close()
    if not args.no_cpu and not only_timed:
        log("cpu baselines ...")
        m_reached = out["config"]["m_reached"]
        out["cpu_baseline"] = cpu_baseline(g, m_reached)
        out["cpu_baselines_more"] = cpu_baselines_more(g, m_reached)
        out["cpu_queue_baselines"] = cpu_queue_baselines()
        if not args.no_graphs:
            # the grid and the road mesh: the full grid; road2048 with the
            # oracle's rounds (its authority, one core); the sequential FIFO
            # and the Jacobi rounds on the same recipe at side 512 (bounded
            # sample: at side 2048 the FIFO form alone takes about a minute)
            out["cpu_graph_baselines"] = cpu_graph_baselines([
                ("grid64", synth.config_graph("grid64"), ("rounds", "fifo", "jacobi")),
                ("road2048", synth.config_graph("road2048"), ("rounds",)),
                ("road512_sample", synth.road(512), ("fifo", "jacobi", "rounds"))],
                budget_s=3.0)
        out["host"] = host_info()
    print(json.dumps(out), flush=True)
    if not parity_ok:
        log("PARITY FAILURE: a timed result differs from the stored oracle result")
        sys.exit(3)


def run_main_legs(args, pkg, torch, dev, g, rec, off, col, w, ctx, q, only_timed):
    dist = torch.empty(g.n, dtype=torch.int64, device=dev)
    pred = torch.empty(g.n, dtype=torch.int32, device=dev)

    # once, outside the timed region: validate the CSR and count reached edges
    ctx.solve(off, col, w, g.src, dist=dist, pred=pred, validate=True)
    reached = (dist != np.iinfo(np.int64).max).cpu().numpy()
    deg = np.diff(g.offsets)
    m_reached = int(deg[reached].sum())
    log(f"reached {int(reached.sum())} vertices, {m_reached} edges")

    if args.calib:
        nbytes = 1 << 30
        a = torch.empty(nbytes // 8, dtype=torch.int64, device=dev)
        b = torch.empty_like(a)
        ms = pkg.probe(0, a, b, size=nbytes, grid=8 * pkg.device_cus(), block=256)
        log(f"calibration copy {nbytes} B in {ms:.3f} ms = {2 * nbytes / ms / 1e6:.0f} GB/s")
        del a, b

    probes = None
    if not args.no_probes and not only_timed:
        probes = run_probes(pkg, torch, dev)
        log(f"probes {probes}")

    # launch shapes, chosen before the timed region: the library's autotuner
    # for the solver, a small search over ticket batch / grid for the queue
    sssp_launch = {}
    tuned = None
    if args.sssp_launch:
        sssp_launch = json.loads(args.sssp_launch)
    elif not args.no_tune and not args.queue_only:
        # the autotuner's pick varies between near-equal shapes from run to
        # run; the timed solve uses a fixed launch from repeated tuning runs
        # (so that the committed kernel profiles are of the timed shape)
        # unless --tune asks for this run's pick
        tuned, tune_ms = ctx.autotune(off, col, w, g.src, reps=5)
        log(f"sssp autotune: {tuned} {tune_ms:.3f} ms")
        sssp_launch = tuned if args.tune or args.scale != 20 else dict(RMAT20_LAUNCH)
    queue_launch = dict(QUEUE_LAUNCH)
    queue_b1_ms = None
    queue_search_best = None
    if args.queue_launch:
        queue_launch = json.loads(args.queue_launch)
    elif not args.sssp_only:
        best = None
        for b in (1, 4, 16, 64, 256):
            for wgsz in (256, 1024):
                for wgs in (64, 256, 0):
                    L = {"ticket_batch": b, "wg_size": wgsz, "wg_count": wgs}
                    t = min(q.bench_mixed(QUEUE_OPS, launch=L)[0]["ms"] for _ in range(2))
                    if b == 1 and (queue_b1_ms is None or t < queue_b1_ms):
                        queue_b1_ms = t
                    if best is None or t < best[0]:
                        best = (t, L)
                if args.no_tune:
                    break
            if args.no_tune:
                break
        queue_search_best = {"launch": best[1], "ms": round(best[0], 4)}
        queue_launch = best[1] if args.tune else dict(QUEUE_LAUNCH)
        log(f"queue search: {best[1]} {best[0]:.3f} ms (b=1 best {queue_b1_ms:.3f} ms); "
            f"timed launch {queue_launch}")
    queue_part = None
    if not only_timed:
        # the partitioned form (one Broker Queue per XCD, Alg. 2's layout)
        queue_part = {}
        for b in (1, 64, 256):
            best = None
            for S in (4, 8):
                L = {"ticket_batch": b, "wg_size": 1024, "wg_count": 0, "segments": S}
                t = min(q.bench_mixed(QUEUE_OPS, launch=L)[0]["ms"] for _ in range(2))
                if best is None or t < best[0]:
                    best = (t, S)
            queue_part[f"b{b}"] = {"mops": round(QUEUE_OPS / (best[0] * 1e-3) / 1e6, 1),
                                   "segments": best[1], "ms": round(best[0], 4)}
        log(f"partitioned queue: {queue_part}")

    def step():
        st = {"ms": float("nan"), "enq_full": 0, "deq_empty": 0}
        if not args.sssp_only:
            st, _, _ = q.bench_mixed(QUEUE_OPS, launch=queue_launch)
        if args.queue_only:
            return st, None
        ctx.solve(off, col, w, g.src, dist=dist, pred=pred, launch=sssp_launch or None)
        return st, ctx.stats()

    for i in range(args.warmup):
        step()
    log(f"warmup {args.warmup} done")
    torch.cuda.synchronize()
    qs, ss = [], []
    t_start = time.perf_counter()
    for i in range(args.steps):
        a_, b_ = step()
        qs.append(a_)
        ss.append(b_)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t_start
    log(f"timed {args.steps} steps in {wall:.3f}s")

    # outside the timed region: the last timed solve's output against the
    # stored result (CPU oracle, certified by the Johnson closed form)
    parity = None
    if rec is not None and not args.queue_only:
        parity = matches_golden(rec, dist, pred) and m_reached == rec["m_reached"]
        log(f"timed output vs stored oracle result: {'exact' if parity else 'MISMATCH'}")

    q_ms = np.array([x["ms"] for x in qs])
    out = {
        "metric": "SSSP GTEPS + queue Mops/s on 1 MI355X; batched/served vs one-at-a-time",
        "value": None, "unit": "GTEPS", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(wall / args.steps * 1e3, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "int64",
        "data": "synthetic",
        "config": {"workload": f"rmat{args.scale}_sssp+queue_mixed", "n": g.n, "m": g.m,
                   "src": g.src, "m_reached": m_reached, "queue_capacity": QUEUE_CAP,
                   "queue_ops": QUEUE_OPS, "parallelism": "single_gpu"},
        "parity": {"rmat20_timed_output": ("exact" if parity else "MISMATCH")
                   if parity is not None else "not checked",
                   "reference": "tests/golden/rmat20.json (CPU oracle, Johnson-certified)"},
    }
    if not args.sssp_only:
        qmops = QUEUE_OPS / (q_ms.mean() * 1e-3) / 1e6
        # one ticket per wave (b = 1, 64 items per ticket) is the queue's
        # design point; the timed launch is the bulk form (64 * b items per
        # ticket, b as in the launch)
        out["queue_mops_b1"] = (round(QUEUE_OPS / (queue_b1_ms * 1e-3) / 1e6, 2)
                                if queue_b1_ms else None)
        out["queue_mops_bulk"] = round(qmops, 2)
        out["queue_mops_bulk_ticket_batch"] = int(queue_launch.get("ticket_batch", 1))
        out["queue_partitioned"] = queue_part
        out["queue"] = {"ms": round(float(q_ms.mean()), 4),
                        "enq_full": int(qs[-1]["enq_full"]),
                        "deq_empty": int(qs[-1]["deq_empty"]), "launch": queue_launch,
                        "search_best": queue_search_best}
        out["queue_roofline"] = queue_roofline(float(q_ms.mean()), queue_launch, queue_b1_ms,
                                               probes)
    if not args.queue_only:
        s_ms = np.array([x["ms"] for x in ss])
        k_ms = np.array([x["solve_ms"] for x in ss])
        gteps = m_reached / (s_ms.mean() * 1e-3) / 1e9
        out["value"] = round(gteps, 4)
        deq = float(np.mean([x["dequeued"] for x in ss]))
        rel = float(np.mean([x["relaxations"] for x in ss]))
        push = float(np.mean([x["pushes"] for x in ss]))
        alg_bytes = BYTES_PER_DEQ * deq + BYTES_PER_EDGE * rel + BYTES_PER_PUSH * push
        achieved = alg_bytes / (k_ms.mean() * 1e-3) / 1e9
        out["launch"] = {"sssp": sssp_launch, "queue": queue_launch,
                         "sssp_autotuner_pick": tuned}
        out["sssp"] = {"ms": round(float(s_ms.mean()), 4),
                       "ms_median": round(float(np.median(s_ms)), 4),
                       "solver_kernel_ms": round(float(k_ms.mean()), 4),
                       "relaxations": int(rel), "dequeued": int(deq), "pushes": int(push),
                       "batches": int(np.mean([x["batches"] for x in ss])),
                       "idle_polls": int(np.mean([x["idle_polls"] for x in ss])),
                       "work_ratio_k": round(rel / m_reached, 3),
                       "relax_per_s_G": round(rel / (k_ms.mean() * 1e-3) / 1e9, 3),
                       "grid": int(ss[-1]["grid"])}
        # the solver kernel of this launch: the sweep form, or with buckets the
        # queue solver's instantiation for 64 * b items per dequeue
        kname = "k_sweep"
        if sssp_launch.get("bucket_width"):
            kname = f"k_solve<{64 * max(1, int(sssp_launch.get('ticket_batch') or 1))}>"

        def counter(path, key):
            # the committed counters were taken at the fixed RMAT-20 launch
            if sssp_launch != RMAT20_LAUNCH:
                return None
            return read_counter_summary(path, kname, key)

        out["roofline"] = {"bound": "hbm", "achieved": round(achieved, 2), "peak": HBM_PEAK_GBS,
                           "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 5),
                           "traffic": counter(PMC_FILE, "hbm_bytes_per_launch"),
                           "kernel": kname,
                           "l2_hit_rate": counter(TCC_FILE, "l2_hit_rate"),
                           "algorithmic_bytes_per_launch": int(alg_bytes),
                           "kernel_ms": round(float(k_ms.mean()), 4)}
        # atomics the solver kernel issues (counter summary of the same
        # sources), per second of its time, against the measured
        # random-atomicMin rate
        n_atomics = counter(TCC_FILE, "TCC_ATOMIC_sum_mean")
        if n_atomics:
            out["atomic_rate_G"] = round(n_atomics / (k_ms.mean() * 1e-3) / 1e9, 3)
        if probes:
            peak = probes.get("atomic_min_rand_8MiB_Gops")
            if peak:
                if n_atomics:
                    out["atomic_frac"] = round(out["atomic_rate_G"] / peak, 4)
                # relaxations are mostly loads (the key check), not atomics
                out["relax_rate_vs_atomic_peak"] = round(
                    (rel / (k_ms.mean() * 1e-3) / 1e9) / peak, 4)
            lpeak = probes.get("load_rand_8MiB_Gops")
            if lpeak:
                # one random coherent key load per relaxation at most
                out["relax_rate_vs_load_peak"] = round(
                    (rel / (k_ms.mean() * 1e-3) / 1e9) / lpeak, 4)
    if probes:
        out["probes"] = probes
    parity_ok = parity is not False
    if only_timed:
        return out, parity_ok

    out["rounds_form"] = rounds_leg(pkg, torch, g, off, col, w, dist, m_reached)
    log(f"rounds form {out['rounds_form']}")
    road_launch = None
    if not args.no_graphs:
        graphs = {}
        # C0: the 64 x 64 grid (latency-bound: a shortest-path tree 128 edges deep)
        graphs["grid64"] = graph_leg(pkg, torch, dev, "grid64", synth.config_graph("grid64"),
                                     reps=20, warmup=10, ctx=ctx)
        log(f"grid64 {graphs['grid64']}")
        # C2 run A: the 2048 x 2048 road mesh; run B: the planted -3 cycle
        road = synth.config_graph("road2048")
        road_launch = road_tune(pkg, torch, dev, road)
        graphs["road2048"] = graph_leg(pkg, torch, dev, "road2048", road, reps=10, warmup=2,
                                       launch=road_launch)
        graphs["road2048_fifo"] = graph_leg(pkg, torch, dev, "road2048", road, reps=3, warmup=1,
                                            launch={"wg_count": 1024, "segments": 8})
        log(f"road2048 {graphs['road2048']}; FIFO order {graphs['road2048_fifo']}")
        del road
        graphs["road2048_negcycle"] = negcycle_leg(pkg, torch, dev,
                                                   synth.config_graph("road2048_negcycle"),
                                                   launch=road_launch)
        log(f"road2048_negcycle {graphs['road2048_negcycle']}")
        out["graphs"] = graphs
        parity_ok &= all(v["parity"] == "exact" for v in graphs.values())
    if not args.no_batched:
        batched = {}
        if args.batched_only in (None, "rmat20x64"):
            srcs = synth.random_sources(g, 64, seed=synth.SEED_BASE + 3)
            bqs = [(off, col, w, int(sv), torch.empty(g.n, dtype=torch.int64, device=dev),
                    torch.empty(g.n, dtype=torch.int32, device=dev)) for sv in srcs]
            blaunch = json.loads(args.batched_launch) if args.batched_launch else None

            def check_x64(queries):
                # all 64 batched answers against the stored per-source results
                gx = golden("rmat20_x64_sources")["queries"]
                ok = all(src == r["src"] and matches_golden(r, d_, p_)
                         for (_, _, _, src, d_, p_), r in zip(queries, gx))
                return "exact (all 64 queries)" if ok else "MISMATCH"

            batched["rmat20_x64_sources"] = batched_leg(
                pkg, torch, dev, "rmat20x64", bqs, [g] * len(bqs), 5, sssp_launch or None,
                blaunch, check=check_x64 if args.scale == 20 else None)
            parity_ok &= batched["rmat20_x64_sources"].get("parity", "exact").startswith("exact")
            log(f"batched rmat20x64 {batched['rmat20_x64_sources']}")
            del bqs
        if args.batched_only in (None, "er256"):
            t0 = time.time()
            ers = synth.er_batch(256)
            log(f"er256 generated in {time.time() - t0:.1f}s")
            bqs = []
            for eg in ers:
                bqs.append((torch.from_numpy(eg.offsets).to(dev),
                            torch.from_numpy(eg.cols).to(dev),
                            torch.from_numpy(eg.w).to(dev), eg.src,
                            torch.empty(eg.n, dtype=torch.int64, device=dev),
                            torch.empty(eg.n, dtype=torch.int32, device=dev)))
            blaunch = json.loads(args.batched_launch) if args.batched_launch else None
            ge = golden("er256")["queries"]
            assert all(graph_sha256(eg) == r["graph_sha256"] and eg.src == r["src"]
                       for eg, r in zip(ers, ge)), "er256: generator output changed"

            def check_er(queries):
                # all 256 batched answers against the stored results
                ok = all(matches_golden(r, d_, p_)
                         for (_, _, _, _, d_, p_), r in zip(queries, ge))
                return "exact (all 256 queries)" if ok else "MISMATCH"

            batched["er256"] = batched_leg(pkg, torch, dev, "er256", bqs, ers, 5, None, blaunch,
                                           check=check_er)
            parity_ok &= batched["er256"]["parity"].startswith("exact")
            log(f"batched er256 {batched['er256']}")
            del bqs, ers
        out["batched"] = batched
    if args.served_requests > 0:
        t0 = time.time()
        # road requests run alone in the batched form (four-wave workgroups):
        # the tuned single-query grid of two-wave workgroups, halved
        rl = None
        if not args.no_graphs and road_launch and road_launch.get("bucket_width"):
            rl = {"bucket_width": int(road_launch["bucket_width"]),
                  "wg_count": max(1, int(road_launch.get("wg_count") or 128) // 2)}
        out["served"] = served_leg(pkg, torch, dev, g, (off, col, w), args.served_requests,
                                   lanes=args.served_lanes, road_launch=rl)
        log(f"served leg in {time.time() - t0:.1f}s: {out['served']}")
        parity_ok &= out["served"]["parity"].startswith("exact")
    out["parity"]["all_checked_legs"] = "exact" if parity_ok else "MISMATCH"
    return out, parity_ok


if __name__ == "__main__":
    main()
