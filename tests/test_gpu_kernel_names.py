"""fc_sampler_kernels: which kernel sampled, where the statistics keep the name of the
sampler whose place it took."""
import pytest

import inputs

pytestmark = pytest.mark.gpu

SMALL = lambda: inputs.barabasi_albert(3000, 3, 1)
CASES = [
    # graph, alpha, asked for, statistics, kernel
    (SMALL, 1.0, None, "wilson_lds", "wilson_jump"),
    (SMALL, 1.0, "lane", "wilson_lane", "wilson_lane"),
    (SMALL, 1.0, "coop", "wilson_coop", "wilson_coop"),
    (SMALL, 1.0, "lds", "wilson_lds", "wilson_lds"),
    (SMALL, 1.0, "hyb", "wilson_hyb", "wilson_hyb"),
    (SMALL, 1.0, "tile", "wilson_tile", "wilson_tile"),
    (lambda: inputs.barabasi_albert(60000, 5, 1), 1.0, None, "wilson_lds", "wilson_lds"),
    (lambda: inputs.rmat(60000, 8, 2), 10.0, None, "wilson_lds", "wilson_hub"),
    (lambda: inputs.rmat(500_000, 8, 2), 1.0, None, "wilson_coop", "wilson_hub"),
    (lambda: inputs.rmat(1_500_000, 8, 2), 1.0, None, "wilson_hyb", "wilson_hub"),
]


@pytest.mark.parametrize("make,alpha,asked,sampler,kernel", CASES)
def test_single_calls(gpu_lib, make, alpha, asked, sampler, kernel):
    dg = gpu_lib.to_device(make())
    st = gpu_lib.sample(dg, alpha=alpha, tree_count=2, sampler=asked)["stats"]
    assert (st["sampler"], st["kernels"]) == (sampler, kernel)
    if dg.n == 3000:
        st = gpu_lib.sample_noalloc(dg, alpha=alpha, tree_count=2, sampler=asked)["stats"]
        assert (st["sampler"], st["kernels"]) == (sampler, kernel)


def test_timed_phases_are_those_of_the_kernel_named(gpu_lib):
    """With option "phase_timing" trees whole in LDS give way to the LDS counters."""
    dg = gpu_lib.to_device(SMALL())
    gpu_lib.set_option("phase_timing", 1)
    try:
        st = gpu_lib.sample(dg, alpha=1.0, tree_count=4)["stats"]
    finally:
        gpu_lib.set_option("phase_timing", 0)
    assert st["kernels"] == "wilson_lds" and sum(st["phase_ms"]) > 0


def test_batches_and_calls_without_trees(gpu_lib):
    graphs = [gpu_lib.to_device(g) for g in (SMALL(), inputs.rmat(400_000, 8, 2), inputs.barabasi_albert(40000, 5, 1))]
    batch = gpu_lib.Batch([{"graph": g, "alpha": 1.0, "tree_count": 2} for g in graphs], seed=1)
    assert batch.run()["kernels"] == "wilson_hub+wilson_lds+wilson_jump"
    assert gpu_lib.sample(graphs[0], alpha=1.0, tree_count=0)["stats"]["kernels"] == ""
