"""Zero right-hand sides with an initial guess: a column whose relative residual has
nothing to be relative to.  The solution is zero; |x| is at most |r| (the smallest
eigenvalue of alpha L + I is 1), which the call reports and keeps below rtol."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

GRAPHS = {
    "star": lambda: inputs.from_edge_list(4073, [(0, i) for i in range(1, 4073)]),
    "tree": lambda: inputs.barabasi_albert(4073, 1, 3),
    "weighted": lambda: inputs.with_weights(inputs.barabasi_albert(3000, 3, 2), 3),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("alpha", [0.01, 3.493104970903123, 1e4])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_zero_column_beside_others(gpu_lib, name, alpha, precision):
    g = GRAPHS[name]()
    r = np.random.default_rng(1)
    B = r.standard_normal((g.n, 8))
    B[:, 3] = 0.0
    X0 = r.standard_normal((g.n, 8))
    out = gpu_lib.solve(g, alpha, B, X0=X0, rtol=1e-9, precision=precision)
    print(name, alpha, precision, out["iters"], out["relres"], flush=True)
    assert np.all(out["relres"] <= 1e-9)
    assert np.isfinite(out["X"]).all()
    assert np.linalg.norm(out["X"][:, 3]) <= 2e-9
    assert out["iters"] < 20000
