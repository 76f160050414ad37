"""Sorting and pair counts where the kernels change: tiles of 1024 and 4096
keys, LDS runs of 1024 and four-way merges above them, keys that differ in few
bytes (even and odd numbers of passes), ties in neither, one or both vectors,
long runs of equal scores, NaN.  Whole numbers: equal to the oracle's, or above
its reach to the all-pairs kernel's, bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _vector(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "distinct":
        return rng.permutation(n).astype(np.float64) / 3.0
    if kind == "few":  # long runs
        return rng.integers(0, 3, n) / 7.0
    return rng.integers(0, max(2, n // 3), n) * 0.1


@pytest.mark.parametrize("n", [2, 63, 64, 65, 257, 1023, 1024, 1025, 2049, 4096, 4097, 9000])
@pytest.mark.parametrize("ka,kb", [("distinct", "distinct"), ("distinct", "some"), ("some", "distinct"),
                                   ("some", "some"), ("few", "some"), ("few", "few")])
def test_kendall_ties_and_widths(gpu_lib, n, ka, kb):
    a, b = _vector(ka, n, n), _vector(kb, n, n + 1)
    assert gpu_lib.kendall_tau(a, b)["counts"] == oracle.kendall_counts(a, b)


@pytest.mark.parametrize("n", [65_536, 65_537, 262_145, (1 << 20) + 1])
@pytest.mark.parametrize("ka,kb", [("few", "some"), ("distinct", "some")])
def test_kendall_equals_all_pairs(gpu_lib, n, ka, kb):
    a, b = _vector(ka, n, 1), _vector(kb, n, 2)
    merge = gpu_lib.kendall_tau(a, b)["counts"]
    gpu_lib.set_option("kendall_pairs", 1)
    try:
        assert merge == gpu_lib.kendall_tau(a, b)["counts"]
    finally:
        gpu_lib.set_option("kendall_pairs", 0)


@pytest.mark.parametrize("n", [1, 1024, 1025, 65_537, 1 << 20, (1 << 20) + 1, (1 << 20) + 4097])
@pytest.mark.parametrize("bytes_", [[], [0], [7], [1, 6], [0, 3, 7], [0, 1, 2, 3, 4, 5, 6]])
def test_rank_by_the_bytes_that_differ(gpu_lib, n, bytes_):
    """Scores whose bits differ in the given bytes only (none: all equal)."""
    rng = np.random.default_rng(n)
    u = np.full(n, np.float64(1.5).view(np.uint64))
    for q in bytes_:
        d = rng.integers(0, 256, n, dtype=np.uint64) if q < 6 else rng.integers(0, 64, n, dtype=np.uint64)
        u ^= d << np.uint64(8 * q)
    s = u.view(np.float64)
    s = np.where(np.isnan(s), 0.5, s)
    order, rank = oracle.ranking(s)
    got = gpu_lib.rank(s)
    assert np.array_equal(got["order"], order) and np.array_equal(got["rank"], rank)


@pytest.mark.parametrize("n,at", [(1, 0), (1025, 1024), (70_000, 35_000)])
def test_nan_writes_nothing(gpu_lib, n, at):
    import ctypes

    import torch
    fc = gpu_lib
    s = torch.arange(n, dtype=torch.float64, device="cuda:0")
    s[at] = float("nan")
    out = torch.full((2, n), -7, dtype=torch.int32, device="cuda:0")
    ctx = fc.context()
    rc = fc.lib().fc_rank(ctx.handle, ctypes.c_void_p(s.data_ptr()), n, 0,
                          ctypes.c_void_p(out[0].data_ptr()), ctypes.c_void_p(out[1].data_ptr()))
    torch.cuda.synchronize()
    assert rc == fc.FC_ERR_ARG and bool((out == -7).all())
    with pytest.raises(fc.FCError) as e:
        fc.kendall_tau(np.arange(n), s)
    assert e.value.code == fc.FC_ERR_ARG
