"""Block CG at the widths and row lengths where its kernels change shape:
columns around one, two and four values a lane and their padding, rows around
the length from which they are summed in segments, right-hand sides that do not
start on 16 bytes, zero and barely nonzero initial guesses.

Bound: every eigenvalue of alpha L + I is at least 1, so |x - x*| <= |r| <=
rtol |b| for each column; the dense binary64 reference adds its own rounding,
below 1e-12 |b| for these condition numbers (at most 1 + 2 alpha d_max w_max)."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RTOL = 1e-10


def _check(fc, g, alpha, k, precision, seed=0, misaligned=False, X0=None):
    import torch
    rng = np.random.default_rng(seed)
    B = rng.standard_normal((g.n, k))
    dev = B
    if misaligned:  # contiguous, on an 8-byte boundary only
        flat = torch.zeros(g.n * k + 1, dtype=torch.float64, device="cuda:0")
        dev = flat[1:].view(g.n, k)
        dev.copy_(torch.from_numpy(B))
        assert dev.data_ptr() % 16 == 8
    out = fc.solve(g, alpha, dev, X0=X0, rtol=RTOL, precision=precision)
    assert (out["relres"] <= RTOL).all()
    w = g.weights if g.weights is not None else np.ones(g.col_idx.size)
    A = np.zeros((g.n, g.n))
    v = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    A[v, g.col_idx] = -alpha * w
    A[np.arange(g.n), np.arange(g.n)] = 1.0 - A.sum(1)
    want = np.linalg.solve(A, B)
    err = np.linalg.norm(out["X"] - want, axis=0) / np.linalg.norm(B, axis=0)
    assert (err <= RTOL + 1e-12).all(), err.max()


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 17, 31, 33, 63, 64])
def test_widths(gpu_lib, precision, k):
    _check(gpu_lib, inputs.barabasi_albert(500, 4, k), 1.0, k, precision, seed=k)
    _check(gpu_lib, inputs.with_weights(inputs.rmat(300, 8, k), 1), 0.5, k, precision, seed=k)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("hub", [127, 128, 129, 255, 256, 257, 1000])
@pytest.mark.parametrize("k", [1, 6, 64])
def test_long_rows(gpu_lib, precision, hub, k):
    """Stars joined by a path: rows just below, at and beyond whole segments."""
    edges, centres, n = [], [], 0
    for leaves in (hub, 3, hub + 128, hub):
        centres.append(n)
        edges += [(n, n + 1 + i) for i in range(leaves)]
        n += leaves + 1
    edges += list(zip(centres[:-1], centres[1:]))
    g = inputs.from_edge_list(n, edges)
    _check(gpu_lib, g, 1.0, k, precision, seed=hub)
    _check(gpu_lib, inputs.with_weights(g, 2), 1.0, k, precision, seed=hub)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("k", [1, 2, 8, 64])
def test_right_hand_sides_on_eight_bytes(gpu_lib, precision, k):
    _check(gpu_lib, inputs.erdos_renyi(400, 0.05, 3), 2.0, k, precision, misaligned=True)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
def test_initial_guess(gpu_lib, precision):
    """A guess that is zero but for its last value is still used (a solution
    given as the guess needs no iteration); isolated vertices; one vertex."""
    fc = gpu_lib
    g = inputs.from_edge_list(1030, [(0, 1), (1, 2), (5, 1029)])
    X0 = np.zeros((g.n, 3))
    X0[-1, -1] = 1e-3
    _check(fc, g, 1.0, 3, precision, X0=X0)
    B = np.zeros((g.n, 1))
    B[1028, 0] = 2.0  # isolated: x = b
    out = fc.solve(g, 1.0, B, X0=B.copy(), rtol=RTOL, precision=precision)
    assert out["iters"] == 0 and np.array_equal(out["X"], B)
    out = fc.solve(inputs.from_edge_list(1, []), 1.0, np.array([[3.0]]), rtol=RTOL, precision=precision)
    assert out["X"][0, 0] == 3.0
