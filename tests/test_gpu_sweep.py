"""GPU parity of the sweep form (sssp_bf, sssp_bf_noalloc) where it can go
wrong: rows at the chunk length, one below and one above it and at its
multiples; batches at the edges of the 64-item, 256-edge and 2048-edge steps;
push buffers that overflow in one sweep; gangs of one workgroup, of a few and
of all; short cycles that improve nothing else. Results are whole numbers and
must equal the oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


def upload(g):
    return (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
            torch.from_numpy(g.w).to(DEV))


def check(g, launch=None):
    print(f"[sweep] {g.name} n={g.n} m={g.m} launch={launch}", flush=True)
    csr = upload(g)
    ctx = pkg.SsspContext(g.n, g.m)
    d, p, neg = ctx.solve(*csr, g.src, launch=launch)
    d1 = torch.empty_like(d)
    p1 = torch.empty_like(p)
    neg1 = pkg.sssp_bf_noalloc(*csr, g.src, d1, p1, launch=launch)
    ctx.close()
    d_ref, p_ref, neg_ref = oracle.sssp(g, method="fifo")
    assert neg == neg1 == neg_ref is False
    for x, ref in ((d, d_ref), (p, p_ref), (d1, d_ref), (p1, p_ref)):
        assert np.array_equal(x.cpu().numpy(), ref)


def rows_of(lengths, seed):
    """Vertex 0 reaches a vertex per length, whose row has that many edges to
    random vertices; potential-shifted weights."""
    rng = np.random.default_rng(seed)
    k = len(lengths)
    n = k + 1 + 3000
    s = np.concatenate([np.zeros(k, np.int64)] +
                       [np.full(x, i + 1, np.int64) for i, x in enumerate(lengths)] +
                       [rng.integers(0, n, 4000)])
    d = np.concatenate([np.arange(1, k + 1), rng.integers(0, n, s.size - k)])
    p = rng.integers(0, 500, n)
    w = rng.integers(1, 300, s.size) + p[s] - p[d]
    return synth.csr_from_edges(n, s, d, w, name="rows", source=0)


@pytest.mark.parametrize("launch", [None, {"wg_count": 1}, {"wg_count": 3, "segments": 2},
                                    {"wg_count": 9, "row_chunk": 64},
                                    {"wg_count": 256, "segments": 8, "row_chunk": 256}])
def test_row_lengths_around_the_chunk(launch):
    lengths = [0, 1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 511, 512, 513, 2047,
               2048, 2049, 4096, 20000]
    check(rows_of(lengths, 11), launch)


@pytest.mark.parametrize("k", [1, 63, 64, 65, 1023, 1025, 5000])
@pytest.mark.parametrize("deg", [1, 32])
def test_sweep_widths(k, deg):
    """A first sweep of one row of k targets, a second of k items whose rows
    hold `deg` edges (64 items x 32 edges fill one 2048-edge step)."""
    check(rows_of([deg] * k, 100 + k + deg), {"wg_count": 1} if k < 1000 else None)


@pytest.mark.parametrize("launch", [{"wg_count": 1}, {"wg_count": 2, "segments": 1}])
def test_push_buffers_overflow(launch):
    """200k vertices on one or two workgroups: a wave improves far more
    vertices in one sweep than its push buffer holds."""
    check(synth.erdos_renyi(200_000, 8, seed=synth.SEED_BASE + 4), launch)


@pytest.mark.parametrize("n", [60, 20_000])
def test_cycle_that_improves_nothing_else(n):
    """A negative 3-cycle behind the last vertex: found and marked without
    waiting for an amount of work."""
    base = synth.potential_random(n, 8 * n, seed=n)
    s, t, w = synth.edges_of(base)
    s = np.concatenate([s, [0, n, n + 1, n + 2]])
    t = np.concatenate([t, [n, n + 1, n + 2, n]])
    w = np.concatenate([w, [5, 2, 2, -5]])
    g = synth.csr_from_edges(n + 3, s, t, w, source=0)
    csr = upload(g)
    ctx = pkg.SsspContext(g.n, g.m)
    assert ctx.solve(*csr, 0)[2]
    d, p, neg = ctx.solve(*csr, 0, neg_inf=True)
    ctx.close()
    d_ref, p_ref, neg_ref = oracle.neg_inf(g)
    assert neg and neg_ref
    assert np.array_equal(d.cpu().numpy(), d_ref) and np.array_equal(p.cpu().numpy(), p_ref)
