"""GPU parity of the small-graph sampler (the automatic choice up to about 26000
vertices) against the CPU oracle, bit for bit: sizes around the widths of waves,
bitmap words, vertices per thread and the largest tree that fits LDS; shallow and
deep forests; cycles longer than an ordinary walk; draw counts that leave 16
bits; every output and entry point that reaches it."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


def _compare(fc, g, alpha, seed, t0, count, stream=0, entry="sample"):
    kw = dict(alpha=alpha, seed=seed, tree_begin=t0, tree_count=count, stream_id=stream, want_visits=True,
              want_digests=True, want_steps=True, want_parents=True, want_tree_visits=True)
    print(f"jump n={g.n} alpha={alpha} seed={seed} trees=[{t0},{t0 + count})", flush=True)
    got = getattr(fc, entry)(fc.to_device(g) if entry == "sample_noalloc" else g, **kw)
    ref = oracle.sample(g, alpha, seed, t0, count, stream=stream, per_tree=True)
    for i in range(count):
        assert np.array_equal(got["parents"][i], ref.parents[i]), f"parents differ in tree {t0 + i}"
        assert np.array_equal(got["tree_visits"][i], ref.tree_visits[i]), f"visits differ in tree {t0 + i}"
    assert np.array_equal(got["tree_digests"], ref.digests)
    assert np.array_equal(got["tree_steps"], ref.steps)
    assert np.array_equal(got["root_counts"], ref.R)
    assert np.array_equal(got["visit_counts"], ref.visits)
    st = got["stats"]
    assert st["sampler"] == "wilson_lds" and st["walk_steps"] == int(ref.steps.sum())
    assert st["roots"] == int(ref.roots.sum())
    return got


@pytest.mark.parametrize("n", [1, 2, 3, 31, 32, 33, 63, 64, 65, 127, 1000, 1023, 1024, 1025, 2049])
def test_sizes(gpu_lib, n):
    g = inputs.erdos_renyi(n, min(1.0, 6.0 / n), n)
    for alpha in (0.3, 5.0):
        _compare(gpu_lib, g, alpha, n, 3, 9, stream=2)
        _compare(gpu_lib, g, alpha, n + 1, 0, 700)


@pytest.mark.parametrize("make,alpha", [
    (lambda: inputs.barabasi_albert(20_000, 5, 1), 1.0),
    (lambda: inputs.rmat(16_384, 8, 2), 10.0),
    (lambda: inputs.rmat(3001, 8, 3), 0.1),
    (lambda: inputs.grid_removed(130, 150, 0.12, 4), 2.0),
    (lambda: inputs.from_edge_list(5000, [(i, i + 1) for i in range(4999)]), 300.0),
    (lambda: inputs.from_edge_list(4001, [(0, i) for i in range(1, 4001)]), 2.0),
    (lambda: inputs.with_weights(inputs.barabasi_albert(9000, 4, 5), 6), 1.0),
], ids=["ba", "rmat", "rmat_iso", "grid", "path", "star", "weighted"])
def test_families(gpu_lib, make, alpha):
    g = make()
    _compare(gpu_lib, g, alpha, 11, 100, 24)
    _compare(gpu_lib, g, alpha, 12, 0, 5, entry="sample_noalloc")


def test_largest_that_fits_and_the_next(gpu_lib):
    """The widest graphs of this sampler (25500 or so; 32 vertices a thread at 1024 threads is
    never reached: 160 KB of LDS end it first) and ones beyond it."""
    for n in (25_000, 25_500, 25_520, 25_600, 26_000, 27_000):
        g = inputs.barabasi_albert(n, 2, n)
        _compare(gpu_lib, g, 1.5, n, 0, 6)


def test_long_cycles(gpu_lib):
    """The first arrows of a complete graph are nearly a random map, whose cycles
    reach sqrt(n): some are longer than an ordinary round follows."""
    n = 3000
    col = np.tile(np.arange(n, dtype=np.int32), (n, 1))
    keep = ~np.eye(n, dtype=bool)
    g = inputs.CSRGraph(n, (np.arange(n + 1) * (n - 1)).astype(np.int32), np.ascontiguousarray(col[keep]))
    _compare(gpu_lib, g, 1.0, 5, 0, 6)


def test_draw_counts_beyond_16_bits(gpu_lib):
    """Heavy edges whose ends are drawn about 10^5 times, beside light ones."""
    edges = [(2 * i, 2 * i + 1, 1.0e5) for i in range(40)] + [(2 * i + 1, 2 * i + 2, 1.0) for i in range(39)]
    g = inputs.from_weighted_edge_list(80, edges)
    got = _compare(gpu_lib, g, 1.0, 7, 0, 6)
    assert int(got["tree_visits"].max()) > 65536 * 2


@pytest.mark.parametrize("threads", [0, 64, 128, 192, 256, 512, 960, 1024])
def test_threads(gpu_lib, threads):
    """Option lds_threads, where it covers the graph with 32 vertices a thread."""
    gpu_lib.set_option("lds_threads", threads)
    try:
        _compare(gpu_lib, inputs.barabasi_albert(2048, 3, 8), 2.0, 3, 0, 40)
        _compare(gpu_lib, inputs.barabasi_albert(2049, 3, 8), 2.0, 3, 0, 40)
        _compare(gpu_lib, inputs.grid_removed(90, 100, 0.1, 8), 1.0, 3, 0, 12)
    finally:
        gpu_lib.set_option("lds_threads", 0)


def test_draw_limit(gpu_lib):
    fc = gpu_lib
    g = inputs.barabasi_albert(3000, 3, 2)
    fc.set_option("max_draws", 2)
    try:
        with pytest.raises(fc.FCError) as e:
            fc.sample(g, alpha=3.0, seed=1, tree_count=20)
        assert e.value.code == fc.FC_ERR_OVERFLOW
    finally:
        fc.set_option("max_draws", 0)
    _compare(fc, g, 3.0, 1, 0, 20)
