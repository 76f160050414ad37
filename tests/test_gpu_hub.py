"""The hubs-first sampler where it can go wrong: sets of one 64-id block up to the
whole graph (a set that fills up, lists that never fit it, 2-cycles and longer
cycles popped from the list), graphs with isolated vertices, hubs and cycles of
three, first arrows drawn ahead and not, weights, a draw limit.  Trees, draw counts
and root counts are integers: they equal the oracle's."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


def _triangles(n):
    e = []
    for i in range(0, n - 2, 3):
        e += [(i, i + 1), (i + 1, i + 2), (i, i + 2)]
    return inputs.from_edge_list(n, e)


def _ring(n):
    return inputs.from_edge_list(n, [(i, i + 1) for i in range(n - 1)] + [(0, n - 1)])


def _star(n, hub):
    return inputs.from_edge_list(n, [(min(i, hub), max(i, hub)) for i in range(n) if i != hub])


GRAPHS = {
    "triangles": (lambda: _triangles(3001), 20.0),
    "ring": (lambda: _ring(3000), 8.0),
    "star": (lambda: _star(400, 37), 1000.0),
    "empty": (lambda: inputs.from_edge_list(130, []), 1.0),
    "ba": (lambda: inputs.barabasi_albert(4000, 4, 1), 2.0),
    "rmat": (lambda: inputs.rmat(4096, 8, 7), 10.0),
    "grid": (lambda: inputs.grid_removed(61, 67, 0.12, 3), 5.0),
    "weighted": (lambda: inputs.with_weights(inputs.barabasi_albert(3000, 3, 2), 3), 3.0),
}


@pytest.fixture
def hub(gpu_lib):
    gpu_lib.set_option("hub", 2)
    gpu_lib.set_option("tile_cross_permille", 0)
    yield gpu_lib
    for name, value in (("hub", 1), ("hub_set", 0), ("hub_threads", 1024), ("predraw_mib", 32768),
                        ("tile_cross_permille", 100), ("max_draws", 0)):
        gpu_lib.set_option(name, value)


def _check(fc, g, alpha, seed, t0, count):
    ref = oracle.sample(g, alpha, seed, t0, count, per_tree=True)
    got = fc.sample(g, alpha=alpha, seed=seed, tree_begin=t0, tree_count=count, want_digests=True,
                    want_steps=True, want_visits=True, want_parents=True, want_tree_visits=True)
    bare = fc.sample(g, alpha=alpha, seed=seed, tree_begin=t0, tree_count=count)
    assert np.array_equal(got["tree_digests"], ref.digests)
    assert np.array_equal(got["tree_steps"], ref.steps)
    assert np.array_equal(got["parents"], ref.parents)
    assert np.array_equal(got["tree_visits"], ref.tree_visits)
    assert np.array_equal(got["visit_counts"], ref.visits)
    assert np.array_equal(got["root_counts"], ref.R)
    assert np.array_equal(bare["root_counts"], ref.R)
    assert got["stats"]["roots"] == int(ref.roots.sum())
    return ref


@pytest.mark.parametrize("size,threads,ahead", [(64, 64, 1), (64, 1024, 0), (256, 128, 0),
                                                (1024, 1024, 1), (2048, 64, 1), (0, 1024, 1)])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_trees_match_oracle(hub, name, size, threads, ahead):
    make, alpha = GRAPHS[name]
    g = make()
    print(f"hubs first {name} n={g.n} set={size} threads={threads} ahead={ahead}", flush=True)
    hub.set_option("hub_set", size)
    hub.set_option("hub_threads", threads)
    hub.set_option("predraw_mib", 32768 if ahead else 0)
    ref = _check(hub, g, alpha, 4, 2, 6)
    if name == "star":
        assert int(ref.tree_visits.max()) > 512


def test_draw_limit(hub):
    g = inputs.barabasi_albert(2000, 3, 1)
    kmax = int(oracle.sample(g, 5.0, 9, 0, 8, per_tree=True).tree_visits.max())
    for size in (64, 0):
        hub.set_option("hub_set", size)
        hub.set_option("max_draws", kmax - 1)
        with pytest.raises(hub.FCError) as e:
            hub.sample(g, alpha=5.0, seed=9, tree_begin=0, tree_count=8)
        assert e.value.code == hub.FC_ERR_OVERFLOW
        hub.set_option("max_draws", kmax)
        _check(hub, g, 5.0, 9, 0, 8)


@pytest.mark.parametrize("n,alpha", [(30000, 1.0), (60000, 10.0)])
def test_default_shape(hub, n, alpha):
    """The shape that the automatic choice takes, on graphs that are larger than a set."""
    hub.set_option("hub", 1)
    _check(hub, inputs.barabasi_albert(n, 5, 1), alpha, 1, 0, 3)
    _check(hub, inputs.rmat(n, 8, 2), alpha, 1, 0, 3)


@pytest.mark.parametrize("size", [64, 0])
def test_batch(hub, size):
    """Jobs of several graphs and alphas in one launch group, run twice."""
    graphs = [inputs.barabasi_albert(4000, 4, 1), inputs.rmat(4096, 8, 7), _triangles(901),
              inputs.with_weights(inputs.barabasi_albert(3000, 3, 2), 3), inputs.from_edge_list(130, [])]
    hub.set_option("hub_set", size)
    jobs = [{"graph": hub.to_device(g), "alpha": al, "tree_count": 5, "stream_id": i, "tree_begin": 3}
            for i, g in enumerate(graphs) for al in (0.5, 6.0)]
    for tune in (False, True):
        batch = hub.Batch(jobs, seed=5, autotune=tune)
        for _ in range(2):
            batch.reset()
            batch.run()
            for k, job in enumerate(jobs):
                ref = oracle.sample(graphs[k // 2], job["alpha"], 5, 3, 5, stream=job["stream_id"])
                got = batch.result(k)["root_counts"]
                assert np.array_equal(got, ref.R), (size, tune, k)


def test_noalloc_holds_what_it_held(hub):
    """A graph whose buffers leave little of the library's static array: the hubs-first
    sampler's would not fit it, the call takes the sampler that does."""
    hub.set_option("hub", 1)
    g = inputs.barabasi_albert(900_000, 1, 3)
    ref = oracle.sample(g, 1.0, 2, 0, 2)
    got = hub.sample_noalloc(hub.to_device(g), 1.0, seed=2, tree_count=2, want_digests=True)
    assert np.array_equal(got["tree_digests"], ref.digests)
    assert np.array_equal(got["root_counts"], ref.R)
    got = hub.sample(g, 1.0, seed=2, tree_count=2, want_digests=True)
    assert np.array_equal(got["tree_digests"], ref.digests)
    assert np.array_equal(got["root_counts"], ref.R)


@pytest.mark.parametrize("name,below,above", [("grid", 1.0, 1.3), ("tree", 9.0, 12.0), ("rmat", 0.05, 5.0)])
def test_both_sides_of_the_rule(hub, name, below, above):
    """Graphs whose in-arrow counts do not fit LDS, where the automatic choice changes from
    hubs first to the other sampler (no hubs; few edges) and where it does not."""
    hub.set_option("hub", 1)
    g = {"grid": lambda: inputs.grid_removed(600, 700, 0.12, 3),
         "tree": lambda: inputs.barabasi_albert(400_000, 1, 1),
         "rmat": lambda: inputs.rmat(700_000, 8, 2)}[name]()
    d = hub.to_device(g)
    for alpha in (below, above):
        ref = oracle.sample(g, alpha, 6, 0, 2, per_tree=True)
        got = hub.sample(g, alpha=alpha, seed=6, tree_count=2, want_digests=True)
        assert np.array_equal(got["tree_digests"], ref.digests)
        assert np.array_equal(got["root_counts"], ref.R)
    batch = hub.Batch([{"graph": d, "alpha": al, "tree_count": 2} for al in (below, above)], seed=6)
    batch.run()
    for k, alpha in enumerate((below, above)):
        assert np.array_equal(batch.result(k)["root_counts"], oracle.sample(g, alpha, 6, 0, 2).R)
