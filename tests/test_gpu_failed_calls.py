"""What calls that fail leave behind and say."""
import ctypes

import numpy as np
import pytest
import torch

import inputs
import oracle

pytestmark = pytest.mark.gpu


def _call(fc, entry, g, trees, alpha=1.0):
    """(return code, statistics as bytes) of a call whose statistics start as 0xAB."""
    ctx = fc.context()
    st = fc.fc_stats()
    ctypes.memset(ctypes.byref(st), 0xAB, ctypes.sizeof(st))
    gs = fc._graph_struct(g)
    ps = fc._params(alpha, seed=3, tau_=max(trees, 1))
    R = torch.zeros(g.n, dtype=torch.int32, device="cuda")
    F = torch.zeros(g.n, dtype=torch.float64, device="cuda")
    rp, fp = fc._ptr(R), fc._ptr(F)
    if entry == "fc_farness":
        rc = fc.lib().fc_farness(ctx.handle, ctypes.byref(gs), ctypes.byref(ps), fp, None, None, rp,
                                 ctypes.byref(st))
    else:
        rc = getattr(fc.lib(), entry)(ctx.handle, ctypes.byref(gs), ctypes.byref(ps), 0, trees, rp, None,
                                      None, None, None, None, ctypes.byref(st))
    return rc, bytes(st), st


@pytest.mark.parametrize("trees", [0, 20])
@pytest.mark.parametrize("n", [700, 40000])
@pytest.mark.parametrize("entry", ["fc_sample", "fc_sample_noalloc", "fc_farness"])
def test_statistics_of_an_unsound_graph_stay_as_they_were(gpu_lib, entry, n, trees):
    """Graphs whose checks are read with the results, and graphs whose checks come first."""
    fc = gpu_lib
    g = inputs.barabasi_albert(n, 3, 1)
    rc, _, st = _call(fc, entry, fc.to_device(g), trees)
    assert rc == fc.FC_OK and st.tau == (max(trees, 1) if entry == "fc_farness" else trees)
    ci = g.col_idx.copy()
    ci[0] = 0  # a loop
    bad = fc.to_device(inputs.CSRGraph(g.n, g.row_ptr, ci))
    rc, raw, _ = _call(fc, entry, bad, trees)
    assert rc == fc.FC_ERR_GRAPH
    assert raw == b"\xab" * len(raw)


def test_a_batch_names_the_limit_of_the_group_that_met_it(gpu_lib):
    """A large graph sampled hubs first (31-bit draw counts) ahead of a small one whose
    whole tree lies in LDS (28 bits): the draw limit is met in the small one alone."""
    fc = gpu_lib
    large = inputs.rmat(400_000, 8, 2)
    small = inputs.from_edge_list(400, [(0, i) for i in range(1, 400)])
    limit = int(oracle.sample(large, 0.05, 5, 0, 2, per_tree=True).tree_visits.max())
    assert int(oracle.sample(small, 1e4, 5, 0, 2, per_tree=True).tree_visits.max()) > limit
    jobs = [{"graph": fc.to_device(large), "alpha": 0.05, "tree_count": 2},
            {"graph": fc.to_device(small), "alpha": 1e4, "tree_count": 2}]
    fc.set_option("max_draws", limit)
    try:
        batch = fc.Batch(jobs, seed=5)
        with pytest.raises(fc.FCError) as e:
            batch.run()
    finally:
        fc.set_option("max_draws", 0)
    assert e.value.code == fc.FC_ERR_OVERFLOW
    assert "2^28 - 1" in str(e.value)
