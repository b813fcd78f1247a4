"""Which form of the solver took a query, as the stats of the call say it, and
that the answer is the oracle's whichever it was, also where solves compete for
the workgroups that a form needs."""
import threading

import numpy as np
import pytest
from scipy.sparse import csr_matrix
from scipy.sparse.csgraph import dijkstra

import oracle
import synth

from test_gpu_strip import csr_of, mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

STRIP, SWEEP, QUEUE = 768, 1024, 128  # threads of a workgroup


def check(g, launch, wg_size):
    print(f"[forms] n={g.n} m={g.m} launch={launch}", flush=True)
    ctx = pkg.SsspContext(g.n, g.m)
    d, p, neg = ctx.solve(*csr_of(g), g.src, launch=launch)
    st = ctx.stats()
    ctx.close()
    d_ref, p_ref, neg_ref = oracle.sssp(g, method="fifo")
    assert neg == neg_ref is False
    assert np.array_equal(d.cpu().numpy(), d_ref)
    assert np.array_equal(p.cpu().numpy(), p_ref)
    assert st["wg_size"] == wg_size
    return st["grid"]


@pytest.mark.parametrize("launch", [None, {"bucket_width": 4}, {"wg_count": 3}])
def test_ids_that_follow_the_mesh_take_strips(launch):
    # 90,000 vertices: 10 strips, 6 of which hold the keys
    grid = check(mesh(300, 300, 30), launch, STRIP)
    assert 6 <= grid <= 10


@pytest.mark.parametrize("launch,wg_size", [(None, SWEEP), ({"bucket_width": 4}, QUEUE)])
def test_ids_that_do_not_follow_it_fall_back(launch, wg_size):
    check(mesh(150, 150, 31, perm=True), launch, wg_size)


@pytest.mark.parametrize("length,launch,wg_size", [
    (699, None, STRIP), (700, None, SWEEP), (30_000, {"bucket_width": 4}, STRIP),
    (30_000, {"bucket_width": 4, "row_chunk": 65536}, STRIP),
    (65, {"row_chunk": 64}, STRIP), (700, {"row_chunk": 4096}, SWEEP)], ids=str)
def test_one_long_row_in_a_mesh(length, launch, wg_size):
    # 90,000 vertices (and 4 edges of the mesh): sweeps take rows of more than 703
    to = np.random.default_rng(36).permutation(90_000)[:length]
    extra = np.stack([np.full(length, 777), to, np.full(length, 500)], 1)
    check(mesh(300, 300, 37, shifted=False, extra=extra), launch, wg_size)


@pytest.mark.parametrize("n,launch,wg_size", [
    (30_000, None, SWEEP), (300_000, None, SWEEP), (60_000, {"bucket_width": 4}, STRIP),
    (300_000, {"bucket_width": 4}, QUEUE)], ids=str)
def test_stars(n, launch, wg_size):
    w = np.random.default_rng(n).integers(1, 1000, n - 1)
    check(synth.csr_from_edges(n, np.zeros(n - 1, np.int64), np.arange(1, n), w, source=0),
          launch, wg_size)


def band(n, reach, degree, seed):
    """Edges to random ids within `reach`."""
    rng = np.random.default_rng(seed)
    s = rng.integers(0, n, int(n * degree))
    t = np.clip(s + rng.integers(-reach, reach + 1, s.size), 0, n - 1)
    return synth.csr_from_edges(n, s, t, rng.integers(1, 1001, s.size), source=n // 2)


@pytest.mark.parametrize("n,reach,degree,launch,wg_size", [
    (100_000, 300, 3, None, STRIP), (100_000, 1000, 5.5, None, STRIP),
    (100_000, 2000, 3, None, SWEEP), (100_000, 4000, 5.5, None, SWEEP),
    (100_000, 100, 3, {"bucket_width": 4}, STRIP), (100_000, 1000, 3, {"bucket_width": 4}, QUEUE),
    (30_000, 2000, 3, {"bucket_width": 4}, STRIP), (30_000, 8000, 3, {"bucket_width": 4}, QUEUE),
    (200_000, 8000, 1.5, None, SWEEP)], ids=str)
def test_ids_within_a_band(n, reach, degree, launch, wg_size):
    # the more edges leave a strip, where neighbourhoods grow fast, the worse
    check(band(n, reach, degree, n + reach), launch, wg_size)


@pytest.mark.parametrize("launch", [None, {"bucket_width": 4}], ids=str)
@pytest.mark.parametrize("dims", [(20, 4096), (8, 64, 64), (4096, 20), (30, 31, 32)], ids=str)
def test_meshes_whose_edges_leave_the_strips(dims, launch):
    # a quarter of a strip's edges and more lead out of it, but rings grow slowly
    i = np.arange(np.prod(dims)).reshape(dims)
    s, t = [], []
    for axis in range(len(dims)):
        a = np.take(i, np.arange(dims[axis] - 1), axis).ravel()
        b = np.take(i, np.arange(1, dims[axis]), axis).ravel()
        s, t = s + [a, b], t + [b, a]
    s, t = np.concatenate(s), np.concatenate(t)
    w = np.random.default_rng(39).integers(1, 1001, s.size)
    check(synth.csr_from_edges(i.size, s, t, w, source=i.size // 2), launch, STRIP)


def test_other_graphs():
    assert check(synth.potential_random(2000, 16000, seed=32), {"wg_count": 9}, SWEEP) == 1
    assert check(synth.potential_random(20000, 160000, seed=33), {"wg_count": 9}, SWEEP) == 9
    check(synth.random_small(100_000, 6_000, 1, 9, 38), None, SWEEP)
    assert check(mesh(60, 60, 34), {"flags": pkg.BQ_F_TRACE, "wg_count": 9}, QUEUE) == 9


def test_contexts_of_small_graphs_hold_a_queue_alone():
    # 2^15 slots in each of 24 queues and half a MiB for the rest; a query that
    # asks for a timeline still runs on it
    n, m, count = 9984, 40960, 40
    free = torch.cuda.mem_get_info()[0]
    ctxs = [pkg.SsspContext(n, m) for _ in range(count)]
    used = (free - torch.cuda.mem_get_info()[0]) / count
    for ctx in ctxs:
        ctx.close()
    assert used <= 8 * 24 * 2**15 + 2**19


def test_every_answer_of_competing_solves():
    # each needs more than half of the CUs for its strips, so at most one at a
    # time gets them
    g = mesh(1500, 1450, 35, shifted=False)
    # weights 1..1000 and distances that float64 holds exactly
    d_ref = dijkstra(csr_matrix((g.w, g.cols, g.offsets), shape=(g.n, g.n)),
                     indices=g.src).astype(np.int64)
    p_ref = oracle.pred(g, d_ref)
    launches = ({"bucket_width": 4}, {"bucket_width": 4, "wg_count": 32})
    got, errors = {}, []

    def work(i):
        try:
            csr, st = csr_of(g), torch.cuda.Stream()
            ctx = pkg.SsspContext(g.n, g.m)
            with torch.cuda.stream(st):
                for j, launch in enumerate(launches):
                    got[i, j] = ctx.solve(*csr, g.src, launch=launch, stream=st)
                st.synchronize()
            ctx.close()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    assert len(got) == 6
    for d, p, neg in got.values():
        assert not neg
        assert np.array_equal(d.cpu().numpy(), d_ref)
        assert np.array_equal(p.cpu().numpy(), p_ref)
