"""The start of a strip solve, on the CPU: a model of the strips' messages in
which a member begins long after the others have sent to it. Keys that the
member fills in by itself give every distance; keys copied from memory, where
the messages are, lose the vertex that a message was for."""
import os
import random
import re

import pytest

INF = 1 << 40
STRIP = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                     "paper_2608_21826_amd", "csrc", "sssp_strip.hpp")


def solve(n, edges, src, members, late, copied, rng):
    """Distances by strips of ceil(n / members) vertices. A key is 2 * label + q;
    member `late` starts once the others have nothing left to do."""
    per = -(-n // members)
    out = [[] for _ in range(n)]
    for u, v, w in edges:
        out[u].append((v, w))
    fresh = [1 if v == src else 2 * INF for v in range(n)]
    mem = [k & ~1 for k in fresh]
    lds = [None] * n
    queue = [[] for _ in range(members)]
    ring = [[] for _ in range(members)]
    started = [False] * members

    def start(r):
        for v in range(r * per, min(n, (r + 1) * per)):
            lds[v] = mem[v] if copied and v != src else fresh[v]
        if src // per == r:
            queue[r].append(src)
        started[r] = True

    def lower(v, cand):
        old, lds[v] = lds[v], min(lds[v], cand)
        if cand < old and old & 1 == 0:
            queue[v // per].append(v)

    def act(r):
        """One message or one vertex; whether there was one."""
        if not started[r]:
            start(r)
            return True
        if ring[r] and (not queue[r] or rng.random() < 0.5):
            v = ring[r].pop(0)
            label, mem[v] = mem[v], mem[v] & ~1
            lower(v, label | 1)
            return True
        if not queue[r]:
            return False
        u = queue[r].pop(rng.randrange(len(queue[r])))
        lds[u] &= ~1
        for v, w in out[u]:
            cand = lds[u] + 2 * w + 1
            if v // per == r:
                lower(v, cand)
            else:
                old, mem[v] = mem[v], min(mem[v], cand)
                if cand < old and old & 1 == 0:
                    ring[v // per].append(v)
        return True

    for held in ((late,), ()):
        busy = True
        while busy:
            order = [r for r in range(members) if r not in held]
            rng.shuffle(order)
            busy = any([act(r) for r in order])
    return [k >> 1 for k in lds]


def reference(n, edges, src):
    d = [INF] * n
    d[src] = 0
    for _ in range(n):
        for u, v, w in edges:
            if d[u] < INF and d[u] + w < d[v]:
                d[v] = d[u] + w
    return d


def path_and_chords(rng):
    n = rng.randrange(6, 30)
    edges = [(u, u + s, rng.randrange(1, 9)) for u in range(n) for s in (1, -1)
             if 0 <= u + s < n]
    edges += [(u, min(n - 1, u + 3), rng.randrange(1, 20)) for u in range(0, n, 4)]
    return n, edges, rng.randrange(n)


@pytest.mark.parametrize("members", [2, 3, 5])
def test_a_member_that_starts_late_loses_nothing(members):
    lost = 0
    for seed in range(60):
        n, edges, src = path_and_chords(random.Random(seed))
        ref = reference(n, edges, src)
        for late in range(members):
            rng = random.Random(seed * 31 + late)
            assert solve(n, edges, src, members, late, False, rng) == ref
            lost += solve(n, edges, src, members, late, True, rng) != ref
    assert lost > 0  # the model tells the two starts apart


def test_the_kernel_fills_its_keys_in():
    # every write of a whole strip's keys in LDS, and none from the keys in memory
    fills = re.findall(r"S\.key\[i\]\s*=(?!=)([^;]*);", open(STRIP).read())
    assert fills
    assert not any("a.key" in f for f in fills)
