"""Long negative cycles in the forms that search for them beside the solve: they
are flagged (or marked) within the launch's time limits, whatever the length of
the cycle and of the rows on it."""
import numpy as np
import pytest
from scipy.sparse import csr_matrix
from scipy.sparse.csgraph import breadth_first_order

import oracle
import synth

from test_gpu_strip import mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")
MINUS_INF = -(1 << 63)


def ring(length, extra=0, seed=1, star=True):
    """A cycle of weight -1 and `length` vertices. star: the source, another vertex
    with the highest id, reaches every vertex of it at distance 1, so that the
    parents close the cycle in the second sweep (equal distances take the
    smaller parent) while every later sweep has few items; `extra` edges per
    vertex of the cycle lead to 5,000 vertices far off; ids are permuted. Without
    star the source is on the cycle and ids follow it."""
    w = np.zeros(length, np.int64)
    w[-1] = -1
    u, v = np.arange(length), np.roll(np.arange(length), -1)
    if not star:
        return synth.csr_from_edges(length, u, v, w, source=0)
    rng = np.random.default_rng(seed)
    sinks, src = length + np.arange(5000), length + 5000
    q = np.concatenate([rng.permutation(length + 5000), [src]])
    s = np.concatenate([u, np.full(length, src), np.repeat(u, extra)])
    t = np.concatenate([v, u, rng.choice(sinks, length * extra)])
    w = np.concatenate([w, np.ones(length), np.full(length * extra, 10**6)])
    return synth.csr_from_edges(src + 1, q[s], q[t], w, source=src)


def check(g, neg_inf, launch=None, entries=("ctx", "noalloc", "batch")):
    print(f"[cycles] n={g.n} m={g.m} neg_inf={neg_inf} launch={launch}", flush=True)
    csr = (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
           torch.from_numpy(g.w).to(DEV))
    ref = np.full(g.n, MINUS_INF)
    # here the cycle reaches all that any edge leads to
    ref[np.setdiff1d(np.arange(g.n), g.cols)] = np.iinfo(np.int64).max
    if g.src not in g.cols:
        ref[g.src] = 0
    for entry in entries:
        d = torch.empty(g.n, dtype=torch.int64, device=DEV)
        p = torch.empty(g.n, dtype=torch.int32, device=DEV)
        if entry == "ctx":
            ctx = pkg.SsspContext(g.n, g.m)
            neg = ctx.solve(*csr, g.src, dist=d, pred=p, launch=launch, neg_inf=neg_inf)[2]
            ctx.close()
        elif entry == "noalloc":
            neg = pkg.sssp_bf_noalloc(*csr, g.src, d, p, launch=launch, neg_inf=neg_inf)
        else:
            batch = pkg.SsspBatch(1, g.n, g.m)
            flags = dict(launch or {}, flags=pkg.BQ_F_NEGINF if neg_inf else 0)
            neg = bool(batch.solve([(*csr, g.src, d, p)], launch=flags)[0])
            batch.close()
        assert neg
        if neg_inf:
            assert np.array_equal(d.cpu().numpy(), ref)
            assert (p.cpu().numpy() == -1).all()


@pytest.mark.parametrize("neg_inf", [False, True])
def test_the_sum_of_a_long_cycle_is_shared_out(neg_inf):
    # adding up this cycle at once takes some 40 ms, while no wait of the other
    # workgroups may last 8 ms (and the whole solve 80 ms)
    check(ring(500, extra=20_000), neg_inf, {"timeout_us": 8_000})


@pytest.mark.parametrize("length", [9000, 20_000, 40_000])
@pytest.mark.parametrize("neg_inf", [False, True])
def test_long_cycles_in_sweeps(length, neg_inf):
    check(ring(length), neg_inf)


@pytest.mark.parametrize("neg_inf", [False, True])
def test_long_cycles_through_many_strips(neg_inf):
    # each strip is busy for one part in 18 to 36 of the solve
    check(ring(300_000, star=False), neg_inf, entries=("ctx", "batch"))


@pytest.mark.parametrize("launch", [None, {"bucket_width": 4}], ids=str)
@pytest.mark.parametrize("neg_inf", [False, True])
@pytest.mark.parametrize("at", [100, 14_000])
def test_a_short_cycle_under_a_crowded_strip(at, neg_inf, launch):
    # three vertices on a cycle of weight -3 reach 60 others each, those 6,000 between
    # them: from the third step on every step holds more vertices than the list. The
    # edge that nothing reaches keeps the labels' lower bound far off
    ring = at + np.arange(3)
    mid = at + 100 + np.arange(180).reshape(3, 60)
    far = 1000 + np.tile(np.arange(6000).reshape(60, 100), (3, 1))
    u = np.concatenate([ring, np.repeat(ring, 60), np.repeat(mid.ravel(), 100)])
    v = np.concatenate([np.roll(ring, -1), mid.ravel(), far.ravel()])
    w = np.concatenate([[-1, -1, -1], np.ones(u.size - 3, np.int64)])
    g = mesh(120, 120, 51, shifted=False, extra=np.stack([u, v, w], 1))
    s, t, x = synth.edges_of(g)
    g = synth.csr_from_edges(g.n + 1, np.append(s, g.n), np.append(t, 0), np.append(x, -10**6),
                             source=at)
    check(g, neg_inf, launch)


@pytest.mark.parametrize("launch", [{}, {"bucket_width": 4}], ids=str)
@pytest.mark.parametrize("neg_inf", [False, True])
def test_a_long_cycle_among_thousands_of_queued_vertices(neg_inf, launch):
    # one strip whose steps hold thousands of vertices: with a move a step a walk goes
    # round this cycle in some hundred ms, and the solve may take 40
    rng = np.random.default_rng(52)
    n, m, length = 15_000, 57_000, 2000
    s, t, w = rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(1, 1001, m)
    p = rng.integers(0, 1001, n)
    c = 3000 + np.arange(length)
    s, t, w = np.append(s, c), np.append(t, np.roll(c, -1)), np.append(w, np.full(length, -1))
    g = synth.csr_from_edges(n, s, t, w + p[s] - p[t], source=int(s[0]))
    csr = [torch.from_numpy(x).to(DEV) for x in (g.offsets, g.cols, g.w)]
    ctx = pkg.SsspContext(g.n, g.m)
    ref = oracle.neg_inf(g, g.src)[0] if neg_inf else None
    for _ in range(3):
        d, _, neg = ctx.solve(*csr, g.src, launch={**launch, "timeout_us": 4000}, neg_inf=neg_inf)
        assert neg
        assert ctx.stats()["wg_size"] == 768
        assert not neg_inf or np.array_equal(d.cpu().numpy(), ref)
    ctx.close()


def hidden_cycle(n, deg, length, seed):
    """A random graph with a cycle of weight -`length` through random vertices, the
    source on it; a random potential hides which edges are negative. Also the marked
    labels: all that the source reaches are on no shortest path."""
    rng = np.random.default_rng(seed)
    s, t, w = (rng.integers(0, n, n * deg), rng.integers(0, n, n * deg),
               rng.integers(1, 1001, n * deg))
    p = rng.integers(0, 1001, n)
    c = rng.permutation(n)[:length]
    s, t, w = np.append(s, c), np.append(t, np.roll(c, -1)), np.append(w, np.full(length, -1))
    g = synth.csr_from_edges(n, s, t, w + p[s] - p[t], source=int(c[0]))
    rows = csr_matrix((np.ones(g.m), g.cols, g.offsets), shape=(n, n))
    ref = np.full(n, np.iinfo(np.int64).max)
    ref[breadth_first_order(rows, g.src, return_predecessors=False)] = MINUS_INF
    return g, ref


def check_hidden(g, ref, neg_inf, timeout_us, wg_size):
    csr = [torch.from_numpy(x).to(DEV) for x in (g.offsets, g.cols, g.w)]
    ctx = pkg.SsspContext(g.n, g.m)
    for _ in range(3):
        d, _, neg = ctx.solve(*csr, g.src, launch={"timeout_us": timeout_us}, neg_inf=neg_inf)
        assert neg
        assert ctx.stats()["wg_size"] == wg_size
        assert not neg_inf or np.array_equal(d.cpu().numpy(), ref)
    ctx.close()
    d = torch.empty(g.n, dtype=torch.int64, device=DEV)
    p = torch.empty(g.n, dtype=torch.int32, device=DEV)
    batch = pkg.SsspBatch(1, g.n, g.m)
    flags = pkg.BQ_F_NEGINF if neg_inf else 0
    assert batch.solve([(*csr, g.src, d, p)], launch={"timeout_us": timeout_us, "flags": flags})[0]
    assert not neg_inf or np.array_equal(d.cpu().numpy(), ref)
    batch.close()


@pytest.mark.parametrize("neg_inf", [False, True])
def test_a_long_cycle_under_wide_sweeps(neg_inf):
    # a walk with a few moves a sweep went round this cycle in 260 to 620 ms; the
    # solve may take 80
    check_hidden(*hidden_cycle(15_000, 8, 8000, 53), neg_inf, 8000, 1024)


@pytest.mark.parametrize("neg_inf", [False, True])
def test_a_long_cycle_in_one_workgroup(neg_inf):
    # 27 to 650 ms with a few moves a sweep; the solve may take 20
    check_hidden(*hidden_cycle(8000, 5, 2000, 54), neg_inf, 2000, 1024)


@pytest.mark.parametrize("count,timeout_us", [(64, 5000), (256, 20_000)])
@pytest.mark.parametrize("neg_inf", [False, True])
def test_long_cycles_in_a_batch_of_small_gangs(count, timeout_us, neg_inf):
    # four workgroups each or one: 150 ms and 550 with a few moves a sweep; the solve
    # may take ten times the limit
    g, ref = hidden_cycle(15_000, 8, 2000, 55)
    csr = [torch.from_numpy(x).to(DEV) for x in (g.offsets, g.cols, g.w)]
    outs = [(torch.empty(g.n, dtype=torch.int64, device=DEV),
             torch.empty(g.n, dtype=torch.int32, device=DEV)) for _ in range(count)]
    batch = pkg.SsspBatch(count, count * g.n, count * g.m)
    flags = pkg.BQ_F_NEGINF if neg_inf else 0
    # each query's graph is its own
    neg = batch.solve([(*[x.clone() for x in csr], g.src, d, p) for d, p in outs],
                      launch={"timeout_us": timeout_us, "flags": flags})
    assert all(neg)
    assert not neg_inf or all(np.array_equal(d.cpu().numpy(), ref) for d, _ in outs)
    batch.close()
