"""Calls that may not allocate what the automatic choice would like (option
"scratch_limit"): the sampler that needs less takes over, on the ids and class offsets
that are its own.  Trees and root counts are integers: they equal the oracle's."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture
def fresh(gpu_lib):
    """The library with a context that holds nothing yet; the session's own comes back."""
    kept = dict(gpu_lib._contexts)
    gpu_lib._contexts.clear()
    yield gpu_lib
    for ctx in gpu_lib._contexts.values():
        ctx.close()
    gpu_lib._contexts.clear()
    gpu_lib._contexts.update(kept)


def _same(fc, g, dg, alpha, trees, refs):
    if alpha not in refs:
        refs[alpha] = oracle.sample(g, alpha, 5, 0, trees)
    got = fc.sample(dg, alpha=alpha, seed=5, tree_count=trees, want_digests=True, want_visits=True)
    assert np.array_equal(got["tree_digests"], refs[alpha].digests)
    assert np.array_equal(got["visit_counts"], refs[alpha].visits)
    assert np.array_equal(got["root_counts"], refs[alpha].R)


@pytest.mark.parametrize("ahead", [True, False])
def test_lds_counters_take_over_on_their_own_ids(fresh, ahead):
    """An R-MAT graph whose counts fit LDS, sampled at an alpha that takes the LDS counters
    and then at one that takes the hubs-first sampler, which gets none, some or all of
    the buffers that only it needs."""
    g = inputs.rmat(30000, 8, 2)
    dg = fresh.to_device(g)
    trees, refs = 8, {}
    fresh.set_option("predraw_mib", 32768 if ahead else 0)
    _same(fresh, g, dg, 0.05, trees, refs)
    for limit in [1] + [q << 19 for q in range(1, 80)]:
        print(f"scratch_limit {limit}", flush=True)
        fresh.set_option("scratch_limit", limit)
        _same(fresh, g, dg, 1.0, trees, refs)
    _same(fresh, g, dg, 0.05, trees, refs)
