"""The small-graph sampler's schedule, modelled on the CPU: 2-cycles popped as
they are found, pointer jumping in place in any order (a jump may read another
one before or after it moved), a stop when a pass settles nobody, and cycles
found from marks that may not stand on a cycle yet.  Tree and arrow counts must
be those of the oracle's sequential walk, whatever the order of the jumps, the
passes before marks are followed and the bound on a walk; rounds that find no
cycle must be followed by one that does.  The model is test code: it shares
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
    full, fulls = False, 0
    while True:
        while listed:
            for v in listed:
                tgt[v] = arrows(v, int(k[v]), t)
                k[v] += 1
                settled[v] = settled[tgt[v]]
            marks = set(listed)
            nxt = []
            for u in listed:
                w = tgt[u]
                if not settled[u] and tgt[w] == u and (w not in marks or u < w):
                    nxt += [u, w]
            assert len(set(nxt)) == len(nxt)
            listed = nxt
        jump = {}
        for v in sorted(opened, key=lambda _: rng.random()):
            settled[v] = settled[v] or settled[tgt[v]]
            jump[v] = n if settled[v] else tgt[v]
        opened = {v for v in opened if jump[v] != n}
        passes = 0
        while opened:
            order = list(opened)
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
            passes += 1
            if not new and passes >= (16 if full else min_passes):
                break
        if not opened:
            return np.array(tgt), k, fulls
        # nobody left can reach u*
        for v in opened:
            seen, x = set(), v
            while x not in seen:
                seen.add(x)
                x = tgt[x]
                assert x != n and not settled[x]
        marks = {jump[v] for v in opened}
        assert marks <= opened
        bound = n + 1 if full else walk
        for c in sorted(marks, key=lambda _: rng.random()):
            x, cyc = tgt[c], [c]
            while x != c and len(cyc) < bound and not (x < c and x in marks):
                cyc.append(x)
                x = tgt[x]
            if x == c:
                listed += cyc
        assert len(set(listed)) == len(listed)
        assert listed or not full
        full = not listed
        fulls += full


CASES = _graphs() + [
    ("ring", inputs.from_edge_list(33, [(i, (i + 1) % 33) for i in range(33)]), 40.0),
    ("triangles", inputs.from_edge_list(30, [(3 * i + a, 3 * i + b) for i in range(10)
                                              for a, b in ((0, 1), (1, 2), (0, 2))]), 9.0),
    ("path", inputs.from_edge_list(40, [(i, i + 1) for i in range(39)]), 30.0),
]


@pytest.mark.parametrize("min_passes,walk", [(5, 64), (1, 64), (1, 2), (16, 1000)])
@pytest.mark.parametrize("name,g,alpha", CASES, ids=[c[0] for c in CASES])
def test_jump_schedule_equals_wilson(name, g, alpha, min_passes, walk):
    seed, stream, t0, count = 0x1234_5678_9ABC, 3, 5, 6
    arrows = _Arrows(g, alpha, seed, stream)
    ref = oracle.sample(g, alpha, seed, t0, count, stream=stream, per_tree=True)
    fulls = 0
    for i in range(count):
        rng = np.random.default_rng([i, min_passes, walk])
        parents, k, f = _jump_tree(g, arrows, t0 + i, rng, min_passes, walk)
        fulls += f
        assert np.array_equal(parents, ref.parents[i]), (name, i)
        assert np.array_equal(k, ref.tree_visits[i]), (name, i)
    if name == "triangles" and walk == 2:
        assert fulls > 0  # walks of two arrows close no triangle: the fallback round ran
