"""The tile sampler's sets in LDS where they can go wrong: more 2-cycles and more
cycle vertices than the list holds, draw counts past the byte kept in LDS, cycles
of three and long paths, tiles of one 64-id block up to the widest, threads that
own 1 to 32 vertices, residuals in LDS and larger than a tile.  Trees, draw counts
and root counts are integers: they equal the oracle's."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


def _edges(n, step):
    return inputs.from_edge_list(n, [(i, i + 1) for i in range(0, n - 1, step)])


def _triangles(n):
    e = []
    for i in range(0, n - 2, 3):
        e += [(i, i + 1), (i + 1, i + 2), (i, i + 2)]
    return inputs.from_edge_list(n, e)


def _star(n, hub):
    return inputs.from_edge_list(n, [(min(i, hub), max(i, hub)) for i in range(n) if i != hub])


GRAPHS = {
    "pairs": (lambda: _edges(3000, 2), 20.0),
    "triangles": (lambda: _triangles(3001), 20.0),
    "path": (lambda: _edges(3000, 1), 5.0),
    "star": (lambda: _star(400, 37), 1000.0),
    "grid": (lambda: inputs.grid_removed(61, 67, 0.12, 3), 5.0),
    "weighted": (lambda: inputs.with_weights(inputs.grid_removed(50, 41, 0.1, 2), 3), 5.0),
}


@pytest.mark.parametrize("tile,threads", [(64, 64), (128, 1024), (1024, 64), (2048, 64), (0, 64),
                                          (0, 1024), (26432, 1024)])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_sets_match_oracle(gpu_lib, name, tile, threads):
    fc = gpu_lib
    make, alpha = GRAPHS[name]
    g = make()
    print(f"tile sets {name} n={g.n} tile={tile} threads={threads}", flush=True)
    ref = oracle.sample(g, alpha, 4, 2, 6, per_tree=True)
    fc.set_option("tile_size", tile)
    fc.set_option("tile_threads", threads)
    try:
        got = fc.sample(g, alpha=alpha, seed=4, tree_begin=2, tree_count=6, want_digests=True,
                        want_visits=True, want_parents=True, want_tree_visits=True, sampler="tile")
        bare = fc.sample(g, alpha=alpha, seed=4, tree_begin=2, tree_count=6, sampler="tile")
    finally:
        fc.set_option("tile_size", 0)
        fc.set_option("tile_threads", 1024)
    assert got["stats"]["sampler"] == "wilson_tile"
    assert np.array_equal(got["tree_digests"], ref.digests)
    assert np.array_equal(got["parents"], ref.parents)
    assert np.array_equal(got["tree_visits"], ref.tree_visits)
    assert np.array_equal(got["visit_counts"], ref.tree_visits.sum(axis=0))
    assert np.array_equal(got["root_counts"], ref.R)
    assert np.array_equal(bare["root_counts"], ref.R)
    if name == "star":
        assert int(ref.tree_visits.max()) > 512


def test_tile_size_limits(gpu_lib):
    """What does not fit six bytes of LDS a vertex stays refused."""
    fc = gpu_lib
    g = inputs.grid_removed(20, 20, 0.1, 2)
    fc.set_option("tile_size", 26496)
    try:
        with pytest.raises(fc.FCError) as e:
            fc.sample(g, alpha=1.0, seed=0, tree_begin=0, tree_count=2, sampler="tile")
        assert e.value.code == fc.FC_ERR_UNSUPPORTED
    finally:
        fc.set_option("tile_size", 0)
