"""The small-graph sampler's schedule, modelled on the CPU: 2-cycles popped as
they are found, pointer jumping in place in any order (a jump may read another
one before or after it moved), a stop when a pass settles nobody, and cycles
found from marks that may not stand on a cycle yet.  Tree and arrow counts must
be those of the oracle's sequential walk, whatever the order of the jumps and
the passes before marks are followed, and the vertices listed exactly those on
cycles.  The model is test code: it shares
nothing with the device kernel."""
import numpy as np
import pytest

import inputs
import oracle
from test_schedule_cpu import _Arrows, _graphs


def _jump_tree(g, arrows, t, rng, min_passes, walk):
    n = g.n
    k = np.ones(n, np.int64)
    tgt = [arrows(v, 0, t) for v in range(n)]
    settled = [w == n for w in tgt] + [True]
    opened = {v for v in range(n) if not settled[v]}
    listed = [v for v in opened if tgt[v] != n and tgt[tgt[v]] == v]
    strays, deeps, wide, again = 0, 0, True, set()
    while True:
        while listed:
            for v in listed:
                tgt[v] = arrows(v, int(k[v]), t)
                k[v] += 1
                again.add(v)
                settled[v] = settled[tgt[v]]
            marks = set(listed)
            nxt = []
            for u in listed:
                w = tgt[u]
                if not settled[u] and tgt[w] == u and (w not in marks or u < w):
                    nxt += [u, w]
            assert len(set(nxt)) == len(nxt)
            listed = nxt
        while True:
            jump, work, deep = {}, set(), False
            for v in sorted(opened, key=lambda _: rng.random()):
                if not settled[v] and not wide and v not in again:
                    continue
                to, steps = tgt[v], 0
                while not wide and not settled[v] and not settled[to] and to not in again:
                    to = tgt[to]
                    steps += 1
                    if steps > walk:
                        deep = True
                        break
                settled[v] = settled[v] or settled[to]
                jump[v] = n if settled[v] else to
                if not settled[v]:
                    work.add(v)
            opened = {v for v in opened if not settled[v]}
            if wide or not deep:
                break
            wide = True
            deeps += 1
        least = min_passes
        while True:
            passes = 0
            while work:
                order = list(work)
                rng.shuffle(order)
                new = False
                held = {}  # jumps read early and written late, as lanes of other waves do
                for v in order:
                    to = jump[jump[v]]
                    if rng.random() < 0.5:
                        held[v] = to
                    else:
                        jump[v] = to
                jump.update(held)
                for v in order:
                    if jump[v] == n:
                        settled[v] = new = True
                        opened.discard(v)
                        work.discard(v)
                passes += 1
                if not new and passes >= least:
                    break
            if not work:
                return np.array(tgt), k, strays, deeps
            # nobody left can reach u*
            for v in work:
                seen, x = set(), v
                while x not in seen:
                    seen.add(x)
                    x = tgt[x]
                    assert x != n and not settled[x]
            marks = {jump[v] for v in work}
            assert marks <= work
            hit, listed = set(), []
            for c in marks:
                x = c
                while True:
                    listed.append(x)
                    x = tgt[x]
                    if x in marks:
                        break
                hit.add(x)
            if hit == marks:
                break
            strays += 1
            least = 1
        assert len(set(listed)) == len(listed)
        wide = False
        rest, alive = {v for v in range(n) if not settled[v]}, True  # exactly the cycle vertices
        while alive:
            held = {tgt[v] for v in rest}
            alive = not rest <= held
            rest &= held
        assert set(listed) == rest


CASES = _graphs() + [
    ("ring", inputs.from_edge_list(33, [(i, (i + 1) % 33) for i in range(33)]), 40.0),
    ("complete", inputs.from_edge_list(60, [(i, j) for i in range(60) for j in range(i)]), 1.0),
    ("path", inputs.from_edge_list(40, [(i, i + 1) for i in range(39)]), 30.0),
]


@pytest.mark.parametrize("min_passes,walk", [(0, 96), (1, 0), (5, 3), (16, 96)])
@pytest.mark.parametrize("name,g,alpha", CASES, ids=[c[0] for c in CASES])
def test_jump_schedule_equals_wilson(name, g, alpha, min_passes, walk):
    seed, stream, t0, count = 0x1234_5678_9ABC, 3, 5, 6
    arrows = _Arrows(g, alpha, seed, stream)
    ref = oracle.sample(g, alpha, seed, t0, count, stream=stream, per_tree=True)
    strays = deeps = 0
    for i in range(count):
        rng = np.random.default_rng([i, min_passes])
        parents, k, s, d = _jump_tree(g, arrows, t0 + i, rng, min_passes, walk)
        strays += s
        deeps += d
        assert np.array_equal(parents, ref.parents[i]), (name, i)
        assert np.array_equal(k, ref.tree_visits[i]), (name, i)
    if name == "complete" and min_passes == 0:
        assert strays > 0  # too few jumps: marks taken back
    if name == "complete" and walk == 0:
        assert deeps > 0  # a walk too long: the round over all unsettled vertices
