"""GPU parity of the one-workgroup solver (sssp_bf, sssp_bf_noalloc on small
graphs) at the edges of its range: vertex counts around a wave, the workgroup
and the LDS limit, edge counts at its limit, long rows that all waves scan
together and more of them than one sweep keeps, every marking and cycle
case. Results are whole numbers and must equal the oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


def both(g, launch=None, neg_inf=False):
    print(f"[small] {g.name} n={g.n} m={g.m} launch={launch} neg_inf={neg_inf}", flush=True)
    csr = (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
           torch.from_numpy(g.w).to(DEV))
    ctx = pkg.SsspContext(g.n, g.m)
    d, p, neg = ctx.solve(*csr, g.src, launch=launch, neg_inf=neg_inf)
    d1, p1 = torch.empty_like(d), torch.empty_like(p)
    neg1 = pkg.sssp_bf_noalloc(*csr, g.src, d1, p1, launch=launch, neg_inf=neg_inf)
    # without predecessors the distances are the same
    d2, none, neg2 = ctx.solve(*csr, g.src, launch=launch, neg_inf=neg_inf, want_pred=False)
    ctx.close()
    assert none is None and neg == neg1 == neg2
    d_ref, p_ref, neg_ref = oracle.neg_inf(g, g.src) if neg_inf else oracle.sssp(g, method="fifo")
    assert neg == neg_ref
    if neg and not neg_inf:
        return
    for x, ref in ((d, d_ref), (p, p_ref), (d1, d_ref), (p1, p_ref), (d2, d_ref)):
        assert np.array_equal(x.cpu().numpy(), ref)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 5119, 5120, 5121])
def test_random_sizes(n):
    both(synth.potential_random(n, 8 * n, seed=n))


@pytest.mark.parametrize("side", [3, 31, 99, 100])  # 100 x 100 is past the limit
def test_meshes_to_the_limit(side):
    both(synth.road(side, plant_cycle=False, seed=side))


@pytest.mark.parametrize("n,m", [(9984, 30000), (9985, 30000), (5000, 40960), (5000, 40961),
                                 (700, 0), (700, 1)])
def test_limits(n, m):
    both(synth.potential_random(n, m, seed=n + m))


def test_long_rows():
    """One row of 9,000 edges, and 200 rows of 190 at the same distance (more
    long rows than a sweep leaves to all waves)."""
    rng = np.random.default_rng(3)
    n = 9500
    s = np.concatenate([np.zeros(200, np.int64), np.repeat(np.arange(1, 201), 150),
                        np.full(9000, 250)])
    d = np.concatenate([np.arange(1, 201), rng.integers(0, n, 30000), rng.integers(0, n, 9000)])
    s, d = np.append(s, 7), np.append(d, 250)
    p = rng.integers(0, 300, n)
    w = np.concatenate([np.full(200, 5), rng.integers(1, 200, s.size - 200)]) + p[s] - p[d]
    both(synth.csr_from_edges(n, s, d, w, name="long", source=0))


@pytest.mark.parametrize("cyc", [1, 2, 5, 400])
@pytest.mark.parametrize("mark", [False, True])
def test_cycles(cyc, mark):
    """A negative cycle with a tail behind a random graph of negative and
    positive weights, found and marked."""
    base = synth.potential_random(1500, 9000, seed=cyc)
    s, t, w = synth.edges_of(base)
    n = base.n
    c = np.arange(n, n + cyc)
    cw = np.full(cyc, 3, dtype=np.int64)
    cw[-1] = -3 * (cyc - 1) - 1
    s = np.concatenate([s, [11], c, [n + cyc - 1]])
    t = np.concatenate([t, [n], np.roll(c, -1), [n + cyc]])
    w = np.concatenate([w, [4], cw, [2]])
    both(synth.csr_from_edges(n + cyc + 1, s, t, w, source=0), neg_inf=mark)
