"""The autotuners return launches of the caller's kind: a kept result of a batch
is for the base launch that it was found with, and what the form that solves
the input does not read comes back as it was given."""
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


def test_gangs_read_no_ticket_batch_queue_or_layout(queries):
    batch, q = queries
    for base in ({}, {"ticket_batch": 2, "flags": pkg.BQ_F_GRAPH}):
        launch, _ = batch.autotune(q, reps=1, base=base)
        for field in ("ticket_batch", "queue_scale", "segments", "flags"):
            assert launch[field] == base.get(field, 0)
        assert 0 < launch["wg_count"] <= pkg.device_cus()


@pytest.mark.parametrize("graph", [synth.potential_random(2000, 16_000, seed=3), synth.road(200)],
                         ids=["small", "mesh"])
@pytest.mark.parametrize("base", [{}, {"ticket_batch": 2, "segments": 3, "wg_count": 16}], ids=str)
def test_one_workgroup_and_strips_read_nothing(graph, base):
    ctx = pkg.SsspContext(graph.n, graph.m)
    launch, ms = ctx.autotune(*upload(graph), graph.src, reps=1, base=base)
    ctx.close()
    assert launch == {**dict.fromkeys(launch, 0), **base}
    assert ms > 0


def test_sweeps_read_no_ticket_batch():
    g = synth.potential_random(30_000, 240_000, seed=4)
    ctx = pkg.SsspContext(g.n, g.m)
    launch, _ = ctx.autotune(*upload(g), g.src, reps=3)
    ctx.close()
    assert launch["bucket_width"] == launch["ticket_batch"] == 0
    assert 0 < launch["wg_count"] <= pkg.device_cus()
