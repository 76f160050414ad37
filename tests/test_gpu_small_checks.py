"""The checks that small graphs get in one launch with their records: each fault, at
the first and last entries and where row offsets lead nowhere; outputs stay as they
were, and the next call on a sound graph is right."""

import numpy as np
import pytest
import torch

import inputs
import oracle

pytestmark = pytest.mark.gpu


def _graph():
    return inputs.barabasi_albert(700, 3, 1)


def _bad(kind):
    g = _graph()
    rp, ci = g.row_ptr.copy(), g.col_idx.copy()
    n, nnz = g.n, int(rp[-1])
    if kind == "first_offset":
        rp[0] = 1
    elif kind == "last_offset":
        rp[-1] = nnz - 1
    elif kind == "negative_offset":
        rp[n // 2] = -5
    elif kind == "huge_offset":
        rp[n // 2] = 2**31 - 1
    elif kind == "all_offsets":
        rp[:] = np.int32(-(2**31))
    elif kind == "falling":
        rp[1:n] = rp[1:n][::-1].copy()
    elif kind == "first_column":
        ci[0] = -1
    elif kind == "last_column":
        ci[-1] = n
    elif kind == "loop":
        ci[0] = 0
    elif kind == "order":
        ci[1], ci[0] = ci[0], ci[1]
    elif kind == "one_way":
        row = 400
        a, b = rp[row], rp[row + 1]
        have = set(ci[a:b].tolist()) | {row}
        lo = ci[a - 1 + 1] if b - a < 2 else ci[a + 1]
        new = [x for x in range(int(ci[a]), int(lo)) if x not in have]
        ci[a] = new[-1] if new else ci[a] - 1
    return g, rp, ci


@pytest.mark.parametrize("kind", ["first_offset", "last_offset", "negative_offset", "huge_offset",
                                  "all_offsets", "falling", "first_column", "last_column", "loop",
                                  "order", "one_way"])
def test_faults(gpu_lib, kind):
    fc = gpu_lib
    g, rp, ci = _bad(kind)
    bad = inputs.CSRGraph(g.n, rp, ci)
    R = torch.full((g.n,), 7, dtype=torch.int32, device="cuda")
    print(f"small checks {kind}", flush=True)
    with pytest.raises(fc.FCError) as e:
        fc.farness(bad, alpha=1.0, tau=20, seed=3)
    assert e.value.code == fc.FC_ERR_GRAPH
    with pytest.raises(fc.FCError) as e:
        fc.sample_noalloc(fc.to_device(bad), 1.0, seed=3, tree_count=20, root_counts=R)
    assert e.value.code == fc.FC_ERR_GRAPH
    assert bool((R == 7).all())
    for count in (0, 20):
        if count == 0:
            with pytest.raises(fc.FCError) as e:
                fc.sample(bad, alpha=1.0, seed=3, tree_count=0)
            assert e.value.code == fc.FC_ERR_GRAPH
            continue
        got = fc.sample(g, alpha=1.0, seed=3, tree_begin=0, tree_count=count)
        assert np.array_equal(got["root_counts"], oracle.sample(g, 1.0, 3, 0, count).R)
