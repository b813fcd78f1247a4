"""Calls between the forms of the solver: batches that hold what several forms
would take, on one workspace in turn, and weights at the limit of the packed
keys in every form that can reach it, each refusal followed by a solve.
Against the oracle; whole numbers, equal."""
import numpy as np
import pytest

import oracle
import synth

from test_gpu_strip import csr_of, mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pkg = pytest.importorskip("paper_2608_21826_amd")

DEV = torch.device("cuda:0")


def outputs(n):
    return (torch.full((n,), -7, dtype=torch.int64, device=DEV),
            torch.full((n,), -7, dtype=torch.int32, device=DEV))


def test_a_crowd_with_other_queries():
    n, count = 1 << 18, 66  # 132 MiB of keys: the batch takes the queue solver
    g = synth.potential_random(n, 6 * n, seed=41)
    others = [mesh(256, 256, 42), mesh(120, 120, 43, perm=True), mesh(30, 30, 44),
              synth.potential_random(20_000, 160_000, seed=45), synth.random_small(1, 0, 1, 9, 46),
              mesh(100, 164, 8, shifted=False, extra=[(9000, 9001, -1500)], source=0)]
    refs = [oracle.sssp(o, method="fifo") for o in others]
    srcs = [g.src] + np.random.default_rng(47).permutation(n)[:count - 1].tolist()
    d0, p0, _ = oracle.sssp(g, method="fifo")
    csr = csr_of(g)
    crowd = [(*csr, int(s), *outputs(n)) for s in srcs]
    rest = [(*csr_of(o), o.src, *outputs(o.n)) for o in others]
    batch = pkg.SsspBatch(count + len(rest), n * count + sum(o.n for o in others),
                          g.m * count + sum(o.m for o in others))
    # the crowd, then gangs, strips and single workgroups, then the crowd again
    for queries, graph in ((rest[:3] + crowd + rest[3:], False), (rest, False), (crowd + rest, True),
                           (rest, True), (crowd + rest, True)):
        for q in queries:
            q[4].fill_(-7)
            q[5].fill_(-7)
        flags = batch.solve(queries, graph=graph)
        for q, flag in zip(queries, flags):
            k = [i for i, r in enumerate(rest) if r[4] is q[4]]
            if not k:
                assert not flag
                continue
            d_ref, p_ref, neg = refs[k[0]]
            assert bool(flag) == neg
            if not neg:
                assert np.array_equal(q[4].cpu().numpy(), d_ref)
                assert np.array_equal(q[5].cpu().numpy(), p_ref)
        if len(queries) > len(rest):
            assert np.array_equal(crowd[0][4].cpu().numpy(), d0)
            assert np.array_equal(crowd[0][5].cpu().numpy(), p0)
    batch.close()
    ctx = pkg.SsspContext(g.n, g.m)
    for _, _, _, s, d, p in crowd:
        d1, p1, neg = ctx.solve(*csr, s)
        assert not neg and torch.equal(d1, d) and torch.equal(p1, p)
    ctx.close()


def at_limit(kind, over):
    """A graph whose n * max |w| is just below (over: at) the limit of its keys,
    2^(62 - shift) with shift = bits of n + 1, plus 1; the largest weight once
    negative, on an edge into a vertex without edges."""
    base = (synth.random_small(40_000, 400_000, 1, 2, 48) if kind == "random"
            else mesh(200, 200, 49, shifted=False, perm=kind == "permuted"))
    n = base.n + 1
    limit = 1 << (62 - (n.bit_length() + 1))
    w = -(-limit // n) if over else (limit - 1) // n
    assert w < 2**31 and (n * w >= limit) == over
    u, v, x = synth.edges_of(base)
    u, v, x = np.append(u, base.src), np.append(v, base.n), np.append(x, 1)
    x = np.where(np.arange(x.size) % 3 == 0, w, x)
    x[-1] = -w
    return synth.csr_from_edges(n, u, v, x, source=base.src)


@pytest.mark.parametrize("kind", ["random", "mesh", "permuted"])
@pytest.mark.parametrize("launch", [None, {"bucket_width": 4}], ids=str)
def test_weights_at_the_limit_of_the_keys(kind, launch):
    below, over = at_limit(kind, False), at_limit(kind, True)
    assert below.n == over.n and below.m == over.m
    d_ref, p_ref, neg_ref = oracle.sssp(below, method="fifo")
    assert not neg_ref
    ctx = pkg.SsspContext(below.n, below.m)
    batch = pkg.SsspBatch(2, 2 * below.n, 2 * below.m)
    cb, co = csr_of(below), csr_of(over)
    (d, p), (d1, p1) = outputs(below.n), outputs(below.n)
    for call in (lambda c, s: ctx.solve(*c, s, dist=d, pred=p, launch=launch)[2],
                 lambda c, s: pkg.sssp_bf_noalloc(*c, s, d, p, launch=launch),
                 lambda c, s: any(batch.solve([(*cb, below.src, d1, p1), (*c, s, d, p)],
                                              launch=launch))):
        for _ in range(2):
            with pytest.raises(pkg.BQError) as e:
                call(co, over.src)
            assert e.value.status == pkg.BQ_ERANGE
            assert not call(cb, below.src)
            assert np.array_equal(d.cpu().numpy(), d_ref)
            assert np.array_equal(p.cpu().numpy(), p_ref)
    assert np.array_equal(d1.cpu().numpy(), d_ref) and np.array_equal(p1.cpu().numpy(), p_ref)
    ctx.close()
    batch.close()
