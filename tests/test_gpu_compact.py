"""GPU tests of the compact column storage (row patterns, x windows): the
automatic schedule must give the same bits as an explicit schedule over the
same layout, which walks the layout's own columns, and stay within tolerance
of the oracle.  The device block of the handle tells which form it keeps."""
import numpy as np
import pytest

from gpu_util import TOL_F32, TOL_F64, check_spmv, dev, host, say, storage_values

import paper_1012_2270_amd as rg
from paper_1012_2270_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg._lib.load()
    return torch


def diagonals(n_rows, n_cols, offsets, dtype=np.float32, seed=1, drop=0.0):
    """Matrix with the given diagonals (column - row), entries outside dropped;
    with drop, whole rows are empty at that rate."""
    rng = np.random.default_rng(seed)
    i = np.arange(n_rows)[:, None] + np.sort(np.asarray(offsets))[None, :]
    keep = (i >= 0) & (i < n_cols) & (rng.random(n_rows) >= drop)[:, None]
    rp = np.zeros(n_rows + 1, np.int64)
    np.cumsum(keep.sum(1), out=rp[1:])
    return W.CSR(n_rows, n_cols, rp, i[keep].astype(np.int32), rng.standard_normal(int(rp[-1])).astype(dtype))


def banded(n, mean, half, seed=2, dtype=np.float32, lo_empty=0.0):
    rng = np.random.default_rng(seed)
    A = W.banded_poisson_matrix(n, mean, half, rng, dtype)
    if lo_empty == 0.0:
        return A
    keep_row = rng.random(n) >= lo_empty
    keep = np.repeat(keep_row, np.diff(A.row_ptr))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.where(keep_row, np.diff(A.row_ptr), 0), out=rp[1:])
    return W.CSR(n, n, rp, A.col[keep], A.val[keep])


def both(oracle, torch, A, vt, sort=1, vec=None, tol=None, **kw):
    """Products of the automatic and of an explicit schedule; device bytes
    the compact form adds."""
    vec = vec or (np.float64 if vt == "f64" else np.float32)
    x = W.uniform_vector(A.n_cols, 3, vec)
    M = rg.rgcsr_from_csr(A, value_dtype=vt, sigma=sort, **kw)
    E = rg.rgcsr_from_csr(A, value_dtype=vt, sigma=sort, pad_loads=0, **kw)
    xd = dev(x)
    bits = np.uint64 if vec == np.float64 else np.uint32
    y, ye = host(M.spmv(xd)), host(E.spmv(xd))
    np.testing.assert_array_equal(y.view(bits), ye.view(bits))
    check_spmv(oracle, A, x, y, vals64=storage_values(oracle, A, vt),
               tol=TOL_F64 if vec == np.float64 else TOL_F32)
    D = rg.rgcsr_from_csr_device(A.n_rows, A.n_cols, dev(A.row_ptr), dev(A.col), dev(A.val),
                                 rg.make_opts(value_dtype=vt, sigma=sort, **kw))
    np.testing.assert_array_equal(host(D.spmv(xd)).view(bits), y.view(bits))
    added = M.info["device_bytes"] - E.info["device_bytes"]
    C = M.clone()
    M.close()
    np.testing.assert_array_equal(host(C.spmv(xd)).view(bits), y.view(bits))
    return added


# widths at the edges of the compiled step counts, ragged last groups
@pytest.mark.parametrize("vt", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("width", [1, 2, 4, 5, 6, 8, 9, 10, 15, 16, 17, 27, 33])
def test_patterns_every_width(torch_cuda, oracle, width, vt):
    n = 5000 + width  # 78 groups and a part of one
    A = diagonals(n, n, np.arange(width) * 7 - 3 * width)
    say("pattern width", width, vt)
    added = both(oracle, torch_cuda, A, vt)
    assert 256 <= added - (n + 255) // 256 * 256 <= 8192 + 256


@pytest.mark.parametrize("kw", [dict(G=128), dict(G=256, sort=512), dict(sort=300), dict(tau=40)])
@pytest.mark.parametrize("shape", [(4100, 4100), (4100, 900), (700, 5000)])
def test_patterns_forms(torch_cuda, oracle, shape, kw):
    """Groups of several wavefronts, reordered rows, rectangular shapes, empty
    rows (all of the rows past the columns among them), FP64 vectors over FP32 values."""
    A = diagonals(*shape, [-900, -31, -1, 0, 1, 30, 1200], drop=0.2)
    say("pattern forms", shape, kw)
    assert both(oracle, torch_cuda, A, "f32", **kw) > 0
    both(oracle, torch_cuda, A, "f32", vec=np.float64, **kw)


def test_patterns_at_the_table_limit(torch_cuda, oracle):
    """255 row lists use one byte each; 257 lists keep the layout's columns."""
    for lists, used in ((255, True), (257, False)):
        n = 64 * 400
        rng = np.random.default_rng(5)
        k = np.arange(n) % lists
        cols = np.sort(np.stack([np.full(n, 0), 1 + k, 400 + k * 3], 1), axis=1) + np.arange(n)[:, None]
        A = W.CSR(n, n + 2000, np.arange(n + 1, dtype=np.int64) * 3, cols.ravel().astype(np.int32),
                  rng.standard_normal(3 * n).astype(np.float32))
        say("pattern lists", lists)
        assert (both(oracle, torch_cuda, A, "f32") > 0) == used


# half bands at the edge of the window (4,096 columns of 256 or 512 rows)
@pytest.mark.parametrize("vt", ["f32", "f64", "f16"])
@pytest.mark.parametrize("mean,half,empty", [(8.0, 200, 0.0), (9.0, 500, 0.02), (30.0, 1900, 0.0), (30.0, 2100, 0.0),
                                             (40.0, 60, 0.3), (3.0, 200, 0.0)])
def test_windows(torch_cuda, oracle, mean, half, empty, vt):
    n = 60_013
    A = banded(n, mean, half, lo_empty=empty)
    say("window", mean, half, empty, vt)
    for sort in (1, 256):
        added = both(oracle, torch_cuda, A, vt, sort=sort)
        # 256 rows (512 of narrow rows with values of at most 4 bytes), sorted within 256
        # unsorted, three nonzeros a row leave more padding than nonzeros
        assert (added > 2 * A.nnz) == (half != 2100 and (mean, sort) != (3.0, 1))


def test_windows_of_a_batch(torch_cuda, oracle):
    """Units that straddle matrices, ragged groups, matrices without entries."""
    torch = torch_cuda
    rng = np.random.default_rng(8)
    mats = [W.banded_poisson_matrix(int(n), 20.0, 300, rng) for n in rng.integers(1, 900, 60)]
    mats.insert(3, W.CSR(130, 70, np.zeros(131, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32)))
    B = rg.rgcsr_from_csr_batch(mats, sigma=256)
    E = rg.rgcsr_from_csr_batch(mats, sigma=256, pad_loads=0)
    assert B.info["device_bytes"] > E.info["device_bytes"] + 2 * B.nnz
    ro, co = B.batch_offsets()
    x = W.uniform_vector(int(co[-1]), 4, np.float32)
    say("window batch", len(mats))
    y = host(B.spmv(dev(x)))
    np.testing.assert_array_equal(y.view(np.uint32), host(E.spmv(dev(x))).view(np.uint32))
    for i, A in enumerate(mats):
        if A.nnz:
            check_spmv(oracle, A, x[co[i]:co[i + 1]], y[ro[i]:ro[i + 1]])


def test_non_finite_x_reaches_only_rows_that_use_it(torch_cuda, oracle):
    for A in (diagonals(9001, 9001, [-64, -1, 0, 1, 64], drop=0.1), banded(9001, 18.0, 300, lo_empty=0.05)):
        x = W.uniform_vector(A.n_cols, 6, np.float32)
        bad = np.array([0, 63, 4000, A.n_cols - 1])
        x[bad] = [np.nan, np.inf, -np.inf, np.nan]
        say("non-finite x")
        y = host(rg.rgcsr_from_csr(A).spmv(dev(x)))
        rows = np.repeat(np.arange(A.n_rows), np.diff(A.row_ptr))
        hit = np.zeros(A.n_rows, bool)
        hit[rows[np.isin(A.col, bad)]] = True
        np.testing.assert_array_equal(np.isfinite(y), ~hit)


def test_values_updated_and_strided_x(torch_cuda, oracle):
    """A value update serves the compact form (it keeps no values); 16-bit
    handles run several right-hand sides as strided single-vector launches."""
    torch = torch_cuda
    for A in (diagonals(5000, 5000, [-70, 0, 70]), banded(9000, 20.0, 400)):
        theta = W.normal_vector(A.nnz, 9, np.float32)
        B = W.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col, theta)
        x = W.uniform_vector(A.n_cols, 10, np.float32)
        M = rg.rgcsr_from_csr(A, keep_csr_map=True)
        rg.rgcsr_set_values(M, dev(theta))
        say("update and strides")
        check_spmv(oracle, B, x, host(M.spmv(dev(x))))
        H = rg.rgcsr_from_csr(A, value_dtype="bf16")
        X = W.uniform_matrix(A.n_cols, 3, 11)
        Y = host(H.spmm(dev(X)))
        for k in range(3):
            check_spmv(oracle, A, X[:, k].copy(), np.ascontiguousarray(Y[:, k]),
                       vals64=storage_values(oracle, A, "bf16"))
