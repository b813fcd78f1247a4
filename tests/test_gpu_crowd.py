"""Batches whose queries share a graph on remapped keys: rows at the edges of
the reordering (a wave, its steps in flight, a workgroup's share, the length
from which a workgroup takes a row), and a batch with so many queries of one
graph that it takes the queue solver. Against the oracle and single solves."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


def csr_of(g):
    return (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
            torch.from_numpy(g.w).to(DEV))


@pytest.mark.parametrize("neg", [False, True])
def test_long_rows_of_a_shared_graph(neg):
    rng = np.random.default_rng(91)
    n = 9000
    deg = rng.integers(0, 9, n)
    deg[rng.permutation(n)[:20]] = [15, 16, 17, 33, 63, 64, 65, 255, 256, 257, 1022, 1023, 1024, 1025, 4095, 4097,
                                    16384, 16385, 20000, 70001]
    u = np.repeat(np.arange(n), deg)
    v = rng.integers(0, n, u.size)
    w = rng.integers(1, 500, u.size)
    g = synth.csr_from_edges(n, u, v, w, source=int(np.argmax(deg)))
    if neg:  # potentials make some weights negative and close no cycle
        p = rng.integers(0, 300, n)
        g = synth.csr_from_edges(n, u, v, w + p[u] - p[v], source=int(np.argmax(deg)))
    srcs = [g.src] + rng.permutation(n)[:3].tolist()
    csr = csr_of(g)
    outs = [(torch.empty(n, dtype=torch.int64, device=DEV),
             torch.empty(n, dtype=torch.int32, device=DEV)) for _ in srcs]
    batch = pkg.SsspBatch(len(srcs), n * len(srcs), g.m * len(srcs))
    for graph in (False, True, True):
        flags = batch.solve([(*csr, int(s), d, p) for s, (d, p) in zip(srcs, outs)],
                            launch={"bucket_width": 64}, graph=graph)
        assert not any(flags)
        for s, (d, p) in zip(srcs, outs):
            d_ref, p_ref, _ = oracle.sssp(g, src=int(s), method="fifo")
            assert np.array_equal(d.cpu().numpy(), d_ref)
            assert np.array_equal(p.cpu().numpy(), p_ref)
    batch.close()


@pytest.mark.parametrize("launch", [None, {"ticket_batch": 1, "row_chunk": 64}])
def test_crowd_on_one_graph(launch):
    n, count = 1 << 18, 66  # 132 MiB of keys
    g = synth.potential_random(n, 6 * n, seed=92)
    csr = csr_of(g)
    srcs = [g.src] + np.random.default_rng(93).permutation(n)[:count - 1].tolist()
    dist = torch.empty((count, n), dtype=torch.int64, device=DEV)
    pred = torch.empty((count, n), dtype=torch.int32, device=DEV)
    batch = pkg.SsspBatch(count, n * count, g.m * count)
    flags = batch.solve([(*csr, int(s), dist[i], pred[i]) for i, s in enumerate(srcs)],
                        launch=launch)
    assert not any(flags)
    batch.close()
    ctx = pkg.SsspContext(g.n, g.m)
    for i, s in enumerate(srcs):
        d, p, neg = ctx.solve(*csr, int(s))
        assert not neg and torch.equal(d, dist[i]) and torch.equal(p, pred[i])
    ctx.close()
    d_ref, p_ref, _ = oracle.sssp(g, src=int(srcs[0]), method="fifo")
    assert np.array_equal(dist[0].cpu().numpy(), d_ref)
    assert np.array_equal(pred[0].cpu().numpy(), p_ref)
