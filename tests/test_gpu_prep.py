"""The preparation kernels: CSR checks, class offsets and the reductions of one call.

The checks are compared with a plain numpy reading of the input contract on
directed graphs that break it in every way, at entry counts around the widths
the kernel works in (64 entries per wave and step, 256 per block, several steps
per lane) and with rows far apart in id."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


def _valid(g):
    """Simple, symmetric, rows strictly ascending (weights equal both ways)."""
    n = g.n
    v = np.repeat(np.arange(n), np.diff(g.row_ptr))
    u = g.col_idx.astype(np.int64)
    if ((u < 0) | (u >= n) | (u == v)).any():
        return False
    if ((v[1:] == v[:-1]) & (u[1:] <= u[:-1])).any():
        return False
    key, rev = v * n + u, u * n + v
    order = np.argsort(rev)
    if not np.array_equal(key, rev[order]):
        return False
    if g.weights is not None:
        w = g.weights
        if not ((w == 0) | ((w >= 2.0 ** -64) & (w <= 2.0 ** 64))).all():
            return False
        return bool((w == w[order]).all())
    return True


def _accepted(fc, g):
    try:
        fc.sample(g, 1.0, seed=1, tree_count=1)
        return True
    except fc.FCError as e:
        assert e.code == fc.FC_ERR_GRAPH
        return False


def _csr(n, v, u, w=None):
    """CSR of the directed entries (v, u) in the order given within each row."""
    order = np.argsort(v, kind="stable")
    row_ptr = np.zeros(n + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(v, minlength=n))
    return inputs.CSRGraph(n, row_ptr, np.asarray(u, np.int32)[order], "", None if w is None else w[order])


def _spread(g, gap):
    """The graph with `gap` - 1 isolated vertices after every vertex."""
    v = np.repeat(np.arange(g.n), np.diff(g.row_ptr)).astype(np.int64)
    return _csr(g.n * gap, v * gap, g.col_idx.astype(np.int64) * gap, g.weights)


def _broken(g, rng):
    """Graphs one change away from g, valid or not as numpy finds them."""
    v = np.repeat(np.arange(g.n), np.diff(g.row_ptr)).astype(np.int64)
    u = g.col_idx.astype(np.int64)
    deg = np.diff(g.row_ptr)
    nnz = u.size
    picks = {0, nnz - 1, 63 % nnz, 64 % nnz, 255 % nnz, 256 % nnz, int(rng.integers(nnz))}
    # an entry of the largest hub and one that points at it
    hub = int(deg.argmax())
    picks |= {int(g.row_ptr[hub]), int(np.flatnonzero(u == hub)[0])}
    w = g.weights
    for j in sorted(picks):
        keep = np.arange(nnz) != j
        yield "no reverse", _csr(g.n, v[keep], u[keep], None if w is None else w[keep])
        for to in (v[j], g.n, -1, (u[j] + 1) % g.n):  # self-loop, out of range, another end
            x = u.copy()
            x[j] = to
            yield f"end {to}", _csr(g.n, v, x, w)
        if j + 1 < nnz and v[j] == v[j + 1]:
            x = u.copy()
            x[[j, j + 1]] = x[[j + 1, j]]
            yield "order", _csr(g.n, v, x, w)
            x = u.copy()
            x[j + 1] = x[j]
            yield "twice", _csr(g.n, v, x, w)
        if w is not None:
            for bad in (w[j] * 2, -1.0, np.nan, 2.0 ** 65):
                x = w.copy()
                x[j] = bad
                yield f"weight {bad}", inputs.CSRGraph(g.n, g.row_ptr, g.col_idx, "", x)


GRAPHS = [("edge", lambda: inputs.from_edge_list(2, [(0, 1)])),
          ("32 edges", lambda: inputs.from_edge_list(33, [(i, i + 1) for i in range(32)])),
          ("star 65", lambda: inputs.from_edge_list(66, [(65, i) for i in range(65)])),
          ("far apart", lambda: _spread(inputs.erdos_renyi(40, 0.2, 3), 1000)),
          ("BA", lambda: inputs.barabasi_albert(700, 3, 1)),
          ("weighted R-MAT", lambda: inputs.with_weights(inputs.rmat(900, 8, 2), 4))]


@pytest.mark.parametrize("name,make", GRAPHS, ids=[n for n, _ in GRAPHS])
def test_graph_checks_against_numpy(gpu_lib, name, make):
    fc = gpu_lib
    g = make()
    assert _valid(g) and _accepted(fc, g)
    seen = set()
    for what, h in _broken(g, np.random.default_rng(5)):
        ok = _valid(h)
        seen.add(ok)
        assert _accepted(fc, h) == ok, f"{name}: {what}"
    assert False in seen


@pytest.mark.parametrize("seed", range(8))
def test_graph_checks_on_directed_graphs(gpu_lib, seed):
    """Directed graphs with as many entries one way as the other (cycles,
    tournaments, pairs of reversed paths) are refused unless symmetric."""
    fc = gpu_lib
    rng = np.random.default_rng(seed)
    n = int(rng.integers(3, 200))
    a = np.arange(n)
    cyc = _csr(n, a, np.roll(a, -1))
    assert not _valid(cyc) and not _accepted(fc, cyc)
    perm = rng.permutation(n)
    tour = rng.random((n, n)) < 0.5
    tour = np.triu(tour, 1) | np.tril(~tour.T, -1)
    v, u = np.nonzero(tour[perm][:, perm])
    g = _csr(n, v, u)
    assert _accepted(fc, g) == _valid(g)
    both = tour | tour.T
    v, u = np.nonzero(both)
    g = _csr(n, v, u)
    assert _valid(g) and _accepted(fc, g)


def test_graph_checks_many_steps_per_lane(gpu_lib):
    """Enough entries for several steps per lane; the last entry broken."""
    fc = gpu_lib
    g = inputs.barabasi_albert(300_000, 8, 2)
    assert g.col_idx.size > 2 * 256 * 4096
    assert _accepted(fc, g)
    for j in (g.col_idx.size - 1, g.col_idx.size // 2 + 33):
        x = g.col_idx.copy()
        x[j] = x[j] + 1 if x[j] + 1 < g.n else x[j] - 1
        h = inputs.CSRGraph(g.n, g.row_ptr, x)
        assert not _valid(h) and not _accepted(fc, h)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1025, 262_145, 1_100_000])
def test_isolated_heavy_graphs_match_the_oracle(gpu_lib, n):
    """Vertex counts around the block widths of the per-vertex passes (64 ids per
    ballot, 1024 per class block, more blocks than one stride covers), most of
    the vertices isolated: records, class offsets and sums feed every output."""
    fc = gpu_lib
    rng = np.random.default_rng(n)
    k = min(n, 300)
    pick = np.sort(rng.choice(n, size=k, replace=False))
    edges = [(int(pick[i]), int(pick[j])) for i in range(k) for j in range(i + 1, k) if rng.random() < 0.05]
    g = inputs.from_edge_list(n, edges)
    ref = oracle.sample(g, 1.0, 3, 0, 2)
    for sampler in ("lds", "hyb", "coop", "tile"):
        if sampler == "lds" and n >= 1 << 18:
            continue  # ids beyond that sampler's width
        got = fc.sample(g, 1.0, seed=3, tree_count=2, want_digests=True, sampler=sampler)
        assert np.array_equal(got["root_counts"], ref.R), sampler
        assert np.array_equal(got["tree_digests"], ref.digests), sampler
    diag, far, clo = oracle.estimate(ref.R, 2)
    out = fc.farness(g, alpha=1.0, seed=3, tau=2)
    assert np.array_equal(out["diag"], diag) and np.array_equal(out["farness"], far)
