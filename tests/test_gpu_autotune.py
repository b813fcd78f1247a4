"""The autotuners return launches of the caller's kind: a kept result of a batch
is for the base launch that it was found with."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


def upload(g):
    return (torch.from_numpy(g.offsets).to(DEV), torch.from_numpy(g.cols).to(DEV),
            torch.from_numpy(g.w).to(DEV))


@pytest.fixture(scope="module")
def queries():
    gs = [synth.potential_random(12_000, 96_000, seed=i) for i in range(2)]
    batch = pkg.SsspBatch(2, sum(g.n for g in gs), sum(g.m for g in gs))
    yield batch, [(*upload(g), g.src, torch.empty(g.n, dtype=torch.int64, device=DEV), None)
                  for g in gs]
    batch.close()


def test_a_kept_batch_launch_is_for_its_base(queries):
    batch, q = queries
    bases = [{"bucket_width": 4}, {}, {"timeout_us": 1_000_000}, {"row_chunk": 64}]
    for base in bases + bases:
        launch, ms = batch.autotune(q, reps=1, base=base)
        assert ms > 0
        for field in ("bucket_width", "timeout_us"):
            assert launch[field] == base.get(field, 0)
