"""GPU parity of the strip form (meshes whose ids follow the mesh): strips of
one to many workgroups with full, short and empty last strips, frontiers beyond
a strip's list, more messages in a step than it stores, rows longer than a lane
scans, cycles inside a strip and across strips, ids that it refuses, and every
entry point that tries it. Results are whole numbers and must equal the
oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


def mesh(rows, cols, seed, shifted=True, extra=(), source=None, perm=False):
    """4-neighbour mesh with random weights (potential-shifted: some negative,
    no negative cycle), extra (u, v, w) edges, row-major or permuted ids."""
    rng = np.random.default_rng(seed)
    n = rows * cols
    idx = np.arange(n).reshape(rows, cols)
    pairs = [(idx[:, :-1], idx[:, 1:]), (idx[:-1], idx[1:])]
    u = np.concatenate([x.ravel() for a, b in pairs for x in (a, b)])
    v = np.concatenate([x.ravel() for a, b in pairs for x in (b, a)])
    w = rng.integers(1, 1001, u.size)
    if shifted:
        p = rng.integers(0, 1001, n)
        w = w + p[u] - p[v]
    if len(extra):
        e = np.asarray(extra)
        u, v, w = (np.concatenate([x, e[:, i]]) for i, x in enumerate((u, v, w)))
    src = int(rng.integers(0, n)) if source is None else source
    if perm:
        q = rng.permutation(n)
        u, v, src = q[u], q[v], int(q[src])
    return synth.csr_from_edges(n, u, v, w, source=src)


def csr_of(g):
    return (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
            torch.from_numpy(g.w).to(DEV))


def check(g, launches=(None,), neg_inf=False):
    print(f"[strip] n={g.n} m={g.m} src={g.src} neg_inf={neg_inf}", flush=True)
    csr = csr_of(g)
    d_ref, p_ref, neg_ref = oracle.neg_inf(g, g.src) if neg_inf else oracle.sssp(g, method="fifo")
    ctx = pkg.SsspContext(g.n, g.m)
    for launch in launches:
        for _ in range(2):
            d, p, neg = ctx.solve(*csr, g.src, launch=launch, neg_inf=neg_inf)
            assert neg == neg_ref
            if not neg or neg_inf:
                assert np.array_equal(d.cpu().numpy(), d_ref)
                assert np.array_equal(p.cpu().numpy(), p_ref)
        d, p = torch.empty_like(d), torch.empty_like(p)
        neg = pkg.sssp_bf_noalloc(*csr, g.src, d, p, launch=launch, neg_inf=neg_inf)
        assert neg == neg_ref
        if not neg or neg_inf:
            assert np.array_equal(d.cpu().numpy(), d_ref)
            assert np.array_equal(p.cpu().numpy(), p_ref)
    ctx.close()


FORMS = (None, {"bucket_width": 4}, {"wg_count": 1}, {"wg_count": 3, "flags": pkg.BQ_F_BWD})


@pytest.mark.parametrize("rows,cols", [(100, 101), (64, 256), (129, 127), (1, 16385), (2, 8193),
                                       (300, 111), (16384, 3)])
@pytest.mark.parametrize("shifted", [False, True])
def test_meshes(rows, cols, shifted):
    check(mesh(rows, cols, rows + cols, shifted), FORMS)


def test_permuted_ids_are_solved_by_the_other_forms():
    check(mesh(120, 120, 5, perm=True), FORMS)


@pytest.mark.parametrize("reach", [6000, 12000])
def test_wide_frontiers_and_long_rows(reach):
    # the source reaches `reach` vertices at once: beyond a strip's list, and in
    # the strips after it beyond the messages of a step
    rows, cols = 150, 200
    src = 4000
    far = src + 1 + np.arange(reach)
    extra = np.stack([np.full(reach, src), far, np.random.default_rng(6).integers(1, 9, reach)], 1)
    check(mesh(rows, cols, 7, extra=extra, source=src), FORMS)


@pytest.mark.parametrize("length,at", [(2, 70), (40, 70), (3, 8100), (300, 8000), (9000, 100)])
@pytest.mark.parametrize("neg_inf", [False, True])
def test_planted_cycles(length, at, neg_inf):
    # a chain of consecutive ids and an edge back that closes a negative cycle,
    # inside a strip or across two and more
    u = at + np.arange(length)
    v = np.roll(u, -1)
    w = np.full(length, -1)
    check(mesh(100, 164, 8, shifted=False, extra=np.stack([u, v, w], 1), source=0),
          FORMS[:2], neg_inf)


@pytest.mark.parametrize("neg_inf", [False, True])
def test_cycle_through_the_source(neg_inf):
    check(mesh(100, 110, 9, shifted=False, extra=[(5000, 5001, -2000)], source=5000), FORMS[:2],
          neg_inf)


def test_unreachable_negative_cycle_is_not_flagged():
    g = mesh(100, 110, 10, shifted=False)
    # ten vertices that nothing reaches, on a negative cycle of their own
    n = g.n + 10
    u = np.repeat(np.arange(g.n), np.diff(g.offsets))
    c = g.n + np.arange(10)
    g2 = synth.csr_from_edges(n, np.concatenate([u, c]), np.concatenate([g.cols, np.roll(c, 1)]),
                              np.concatenate([g.w, np.full(10, -3)]), source=g.src)
    check(g2, FORMS)


def test_weights_of_zero_and_range_limits():
    g = mesh(100, 110, 11, shifted=False)
    for w in (np.zeros(g.m), np.full(g.m, 2**31 - 1)):
        check(synth.csr_from_edges(g.n, np.repeat(np.arange(g.n), np.diff(g.offsets)), g.cols, w,
                                   source=g.src))


def test_watchdog_then_a_solve():
    g = mesh(300, 300, 12)
    csr = csr_of(g)
    ctx = pkg.SsspContext(g.n, g.m)
    for launch in ({}, {"bucket_width": 4}):
        with pytest.raises(pkg.BQError) as ei:
            ctx.solve(*csr, g.src, launch={**launch, "timeout_us": 1})
        assert ei.value.status == pkg.BQ_ETIMEOUT
        d, _, _ = ctx.solve(*csr, g.src, launch=launch)
        assert np.array_equal(d.cpu().numpy(), oracle.sssp(g, method="fifo")[0])
    ctx.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batches(graph):
    gs = [mesh(100, 120, 13), mesh(256, 256, 14), mesh(120, 120, 15, perm=True),
          synth.potential_random(20000, 160000, seed=16), mesh(30, 30, 17),
          mesh(100, 164, 8, shifted=False, extra=[(9000, 9001, -1500)], source=0)]
    outs = [(torch.empty(g.n, dtype=torch.int64, device=DEV),
             torch.empty(g.n, dtype=torch.int32, device=DEV)) for g in gs]
    batch = pkg.SsspBatch(len(gs), sum(g.n for g in gs), sum(g.m for g in gs))
    q = [(*csr_of(g), g.src, d, p) for g, (d, p) in zip(gs, outs)]
    for launch in (None, None, {"wg_count": 4}):
        flags = batch.solve(q, launch=launch, graph=graph)
        for g, (d, p), flag in zip(gs, outs, flags):
            d_ref, p_ref, neg = oracle.sssp(g, method="fifo")
            assert bool(flag) == neg
            if not neg:
                assert np.array_equal(d.cpu().numpy(), d_ref)
                assert np.array_equal(p.cpu().numpy(), p_ref)
    batch.close()


def test_solves_that_compete_for_the_chip():
    # each needs more than half of the CUs for its strips: at most one at a time
    # gets them, the others wait their time out and take the other forms
    import threading
    gs = [mesh(1500, 1450, 20 + i, shifted=False) for i in range(3)]
    got, errors = [None] * 3, []

    def work(i):
        try:
            csr, st = csr_of(gs[i]), torch.cuda.Stream()
            ctx = pkg.SsspContext(gs[i].n, gs[i].m)
            with torch.cuda.stream(st):
                for launch in ({"bucket_width": 4}, {"bucket_width": 4, "wg_count": 32}):
                    d, p, neg = ctx.solve(*csr, gs[i].src, launch=launch, stream=st)
                    assert not neg
                    got[i] = (d.cpu().numpy(), p.cpu().numpy())
            ctx.close()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for i in range(3):  # alone, in strips
        ctx = pkg.SsspContext(gs[i].n, gs[i].m)
        d, p, _ = ctx.solve(*csr_of(gs[i]), gs[i].src)
        ctx.close()
        assert np.array_equal(d.cpu().numpy(), got[i][0])
        assert np.array_equal(p.cpu().numpy(), got[i][1])
