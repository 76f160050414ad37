"""First arrows ahead on both sides of the entries from which rows wait in LDS, with one
tree, a group of trees and one more: trees are integers and equal the oracle's."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(104_000, 5), (106_000, 5), (60_000, 12)])
@pytest.mark.parametrize("trees", [1, 16, 33])
def test_rows_in_lds_and_not(gpu_lib, n, m, trees):
    g = inputs.barabasi_albert(n, m, 3)
    print(f"first arrows n={n} nnz={g.col_idx.size} trees={trees}", flush=True)
    ref = oracle.sample(g, 0.5, 11, 5, trees, per_tree=True)
    got = gpu_lib.sample(g, alpha=0.5, seed=11, tree_begin=5, tree_count=trees, want_digests=True)
    assert got["stats"]["sampler"] == "wilson_lds" and got["stats"]["ms_predraw"] > 0.0
    assert np.array_equal(got["tree_digests"], ref.digests)
    assert np.array_equal(got["root_counts"], ref.R)
