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
