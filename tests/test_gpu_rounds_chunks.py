"""The round form at the edges of its chunks: edge counts around a slice of 64,
the eight slices that a wave keeps in flight and a wave's chunk, on rings that
wrap at every offset. Distances, predecessors and the flag must equal the
oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("launch", [
    None, {"wg_size": 64, "wg_count": 1, "ticket_batch": 9},
    {"wg_size": 64, "wg_count": 2, "ticket_batch": 8, "flags": pkg.BQ_F_BWD},
    {"wg_size": 128, "wg_count": 1, "ticket_batch": 64},
])
@pytest.mark.parametrize("m", [1, 63, 64, 65, 511, 512, 513, 575, 577, 1024, 1087, 4097])
def test_chunk_edges(m, launch):
    rng = np.random.default_rng(m)
    n = max(2, m // 4)
    u, v = rng.integers(0, n, (2, m))
    g = synth.csr_from_edges(n, u, v, rng.integers(0, 40, m))
    print(f"[chunks] n={n} m={m} launch={launch}", flush=True)
    ctx = pkg.RoundsContext(g.n, g.m)
    csr = (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
           torch.from_numpy(g.w).to(DEV))
    d_ref, p_ref, _ = oracle.sssp(g, method="fifo")
    for _ in range(3):
        d, p, neg = ctx.solve(*csr, g.src, launch=launch)
        assert not neg
        assert np.array_equal(d.cpu().numpy(), d_ref) and np.array_equal(p.cpu().numpy(), p_ref)
    ctx.close()
