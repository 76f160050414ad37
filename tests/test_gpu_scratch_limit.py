"""Calls that may not allocate what the automatic choice would like (option
"scratch_limit"): the sampler that needs less takes over, on the ids and class offsets
that are its own.  Trees and root counts are integers: they equal the oracle's."""
import numpy as np
import pytest
import torch

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


def _runs(fc, limit, calls):
    """Whether a context that may hold `limit` bytes serves `calls`; they are checked."""
    for ctx in fc._contexts.values():
        ctx.close()
    fc._contexts.clear()
    fc.set_option("scratch_limit", limit)
    try:
        calls()
    except fc.FCError as e:
        assert e.code == fc.FC_ERR_NOMEM
        return False
    return True


def _least(fc, calls, upto, step=1 << 16):
    """The least limit (to `step` bytes) at which `calls` are served."""
    lo, hi = 0, upto // step
    assert _runs(fc, upto, calls)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if _runs(fc, mid * step, calls):
            hi = mid
        else:
            lo = mid
    return hi * step


@pytest.mark.parametrize("n,trees", [(30000, 64), (400_000, 8), (1_500_000, 2)])
def test_hubs_first_needs_no_more_than_the_sampler_it_replaces(fresh, n, trees):
    """R-MAT graphs for which hubs first takes the place of the LDS counters, the global
    counters and the hybrid: what these fit is served, with the right trees, and so is
    everything above (where hubs first gets some of its buffers, then all of them)."""
    g = inputs.rmat(n, 8, 2)
    dg = fresh.to_device(g)
    refs = {}

    def replaced():
        fresh.set_option("hub", 0)
        fresh.sample(dg, alpha=1.0, seed=5, tree_count=trees)

    least = _least(fresh, replaced, 8 << 30)
    print(f"n={n} least {least}", flush=True)
    for percent in range(100, 200, 6):
        # (64 KiB: the counts by which the choice is made)
        limit = least * percent // 100 + (1 << 16)
        assert _runs(fresh, limit, lambda: _same(fresh, g, dg, 1.0, trees, refs)), (least, percent)


def test_earlier_arrows_give_way(fresh):
    """Pre-drawn arrows that an earlier call left do not stand in a later call's way."""
    small, large = inputs.rmat(30000, 8, 2), inputs.rmat(400_000, 8, 2)
    ds, dl = fresh.to_device(small), fresh.to_device(large)

    def calls(mib):
        fresh.set_option("hub", 1)
        fresh.set_option("predraw_mib", mib)
        fresh.sample(ds, alpha=1.0, seed=5, tree_count=512)
        fresh.set_option("hub", 0)
        fresh.sample(dl, alpha=1.0, seed=5, tree_count=8)

    # without arrows ahead the first call keeps them in its slots
    least = _least(fresh, lambda: calls(0), 8 << 30)
    assert _runs(fresh, least + (1 << 16), lambda: calls(32768))


@pytest.mark.parametrize("tune", [False, True])
def test_batches_need_no_more_than_without_hubs_first(fresh, tune):
    """Jobs on graphs for which hubs first takes the place of the LDS and of the global
    counters, and a small one beside them."""
    graphs = [inputs.rmat(400_000, 8, 2), inputs.rmat(30000, 8, 2), inputs.barabasi_albert(3000, 3, 1)]
    on_device = [fresh.to_device(g) for g in graphs]
    refs = [oracle.sample(g, 1.0, 5, 0, 2).R for g in graphs]

    def create(hub):
        fresh.set_option("hub", hub)
        batch = fresh.Batch([{"graph": d, "alpha": 1.0, "tree_count": 2} for d in on_device], seed=5,
                            autotune=tune)
        batch.run()
        got = [batch.result(k)["root_counts"] for k in range(len(graphs))]
        batch.close()
        assert all(np.array_equal(a, b) for a, b in zip(got, refs))

    least = _least(fresh, lambda: create(0), 8 << 30)
    print(f"least {least}", flush=True)
    for percent in range(100, 200, 9):
        assert _runs(fresh, least * percent // 100 + (1 << 16), lambda: create(1)), (least, percent)


@pytest.mark.parametrize("precision,size,k", [("fp32_refined", 4, 5), ("fp32_refined", 4, 3), ("fp64", 8, 3)])
def test_solver_needs_no_more_than_six_vectors(fresh, precision, size, k):
    """Columns are padded to whole 16-byte loads where there is room.  Without it the inner
    vectors have k columns: the least limit is that of the residual, five vectors in the
    inner precision and the partial sums, and the solution the same to the tolerance."""
    g = inputs.grid_removed(300, 300, 0.12, 3)
    dg = fresh.to_device(g)
    B = np.random.default_rng(1).standard_normal((g.n, k))
    got = {}

    def call():
        got["x"] = fresh.solve(dg, 1.0, B, rtol=1e-9, precision=precision)

    assert _runs(fresh, 1 << 30, call)
    full = got["x"]
    least = _least(fresh, call, 1 << 30)
    print(f"least {least}", flush=True)
    partials = 2 * 8 * 64 * max(64, 8 * torch.cuda.get_device_properties(0).multi_processor_count)
    assert least <= 8 * g.n * k + 5 * size * g.n * k + partials + (1 << 17)
    assert _runs(fresh, least, call)
    assert float(got["x"]["relres"].max()) <= 1e-9
    # both solve a system whose smallest eigenvalue is 1: they are as close as their residuals
    norm = np.linalg.norm(B, axis=0)
    assert np.all(np.linalg.norm(got["x"]["X"] - full["X"], axis=0) <= 2e-9 * norm)
