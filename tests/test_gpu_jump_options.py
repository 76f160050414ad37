"""Launch options of the small-graph sampler."""
import numpy as np
import pytest
import torch

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_cu", [1, 2])
def test_workgroups_per_cu_are_capped(gpu_lib, per_cu):
    """Option "lds_wg_per_cu", which a small graph obeyed with LDS counters too."""
    g = inputs.erdos_renyi(1000, 0.01, 0)
    dg = gpu_lib.to_device(g)
    most = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    trees = 4096
    ref = oracle.sample(g, 1.0, 3, 0, trees)
    gpu_lib.set_option("lds_wg_per_cu", per_cu)
    try:
        got = gpu_lib.sample(dg, alpha=1.0, seed=3, tree_count=trees)
        batch = gpu_lib.Batch([{"graph": dg, "alpha": 1.0, "tree_count": trees}], seed=3)
        st = batch.run()
    finally:
        gpu_lib.set_option("lds_wg_per_cu", 0)
    assert np.array_equal(got["root_counts"], ref.R)
    assert np.array_equal(batch.result(0)["root_counts"], ref.R)
    assert got["stats"]["trees_in_flight"] == most
    assert st["trees_in_flight"] == most
