"""Long negative cycles in the forms that search for them beside the solve: they
are flagged (or marked) within the launch's time limits, whatever the length of
the cycle and of the rows on it."""
import numpy as np
import pytest

import synth

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
    if g.src == g.n - 1:
        ref[g.src] = 0  # no edge leads back to the source
        ref[np.setdiff1d(np.arange(g.n - 1), g.cols)] = np.iinfo(np.int64).max
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
