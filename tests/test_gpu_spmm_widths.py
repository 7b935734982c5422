"""GPU tests of the SpMM of any width: every k from 2 to 33 and some above,
leading dimensions and bases at any element, long rows of every item kind,
row patterns, reordered and empty rows, small groups, batches; each column
against the oracle within the FP32 / FP64 tolerances, the columns behind k
untouched, and (grouped rows only) the bits of the single-column launches."""
import numpy as np
import pytest

from gpu_util import TOL_F32, TOL_F64, dev, host, say

import paper_1012_2270_amd as rg
from paper_1012_2270_amd import _lib
from paper_1012_2270_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg._lib.load()
    return torch


def product(torch, M, X, k, ldy, off):
    """Y = A X through the C ABI on blocks that start `off` elements into their
    buffers, Y filled with a marker first."""
    n, ldx = X.shape
    xb = torch.zeros(n * ldx + off, dtype=X.dtype, device="cuda:0")
    xb[off:] = X.reshape(-1)
    yb = torch.full((M.n_rows * ldy + off,), 77.0, dtype=X.dtype, device="cuda:0")
    es = X.element_size()
    _lib.call("rgcsr_spmv_batched", M.handle, k, xb.data_ptr() + off * es, ldx, yb.data_ptr() + off * es, ldy,
              rg._code_of_tensor(X), 0, torch.cuda.current_stream().cuda_stream)
    return host(yb)[off:].reshape(M.n_rows, ldy)


def check(oracle, torch, A, M, k, dtype, pad=0, off=0, bits=False):
    Xh = W.uniform_matrix(A.n_cols, k + pad, 50 + k, dtype)
    X = dev(Xh)
    Y = product(torch, M, X, k, k + pad, off)
    assert np.all(Y[:, k:] == 77.0)
    ref = oracle.csr_spmm(A, np.ascontiguousarray(Xh[:, :k]))
    for c in {0, k // 2, k - 2, k - 1}:
        s = oracle.csr_absmv(A, Xh[:, c].copy())
        e = oracle.scaled_error(np.ascontiguousarray(Y[:, c]), ref[:, c], s)
        assert e <= (TOL_F64 if dtype == np.float64 else TOL_F32), (k, c, e)
        if bits:
            y1 = host(M.spmv(X[:, c].contiguous()))
            np.testing.assert_array_equal(y1.view(np.uint8), np.ascontiguousarray(Y[:, c]).view(np.uint8))


@pytest.mark.parametrize("vt,vec", [("f32", np.float32), ("f64", np.float64), ("f32", np.float64)])
@pytest.mark.parametrize("kind", ["patterns", "short", "long"])
def test_every_width(torch_cuda, oracle, kind, vt, vec):
    torch = torch_cuda
    if kind == "patterns":
        A, lay = W.laplacian_2d_5pt(50, dtype=np.float64), dict()
    elif kind == "short":
        A, lay = W.random_csr(2500, 1900, seed=3, max_len=14, empty_frac=0.2), dict(sigma=300)
    else:
        A = W.random_csr(900, 40_000, seed=4, max_len=200, long_rows=6, long_len=20_000)
        lay = dict(sigma=64, tau=10)
    if vt == "f32":
        A = A.astype(np.float32)
    M = rg.rgcsr_from_csr(A, value_dtype=vt, **lay)
    for k in list(range(2, 34)) + [40, 65]:
        say("spmm width", kind, vt, vec.__name__, k)
        check(oracle, torch, A, M, k, vec, pad=k % 3, off=k % 5, bits=kind != "long" and k % 4 == 3)


@pytest.mark.parametrize("lay", [dict(G=16), dict(G=128, sigma=256), dict(G=64, pad_loads=2), dict(G=32, tau=6)])
def test_group_sizes(torch_cuda, oracle, lay):
    A = W.random_csr(1500, 1500, seed=6, max_len=12, empty_frac=0.0, dtype=np.float32)
    M = rg.rgcsr_from_csr(A, **lay)
    for k in (2, 3, 5, 8, 13, 24, 32):
        say("spmm groups", lay, k)
        check(oracle, torch_cuda, A, M, k, np.float32, pad=1)


def test_batch_panels_and_non_finite(torch_cuda, oracle):
    torch = torch_cuda
    mats = [W.random_csr(300 + 37 * i, 200 + 51 * i, seed=30 + i, max_len=9, dtype=np.float32) for i in range(5)]
    B = rg.rgcsr_from_csr_batch(mats, sigma=128)
    ro, co = B.batch_offsets()
    for k in (3, 7, 18):
        say("spmm batch", k)
        X = W.uniform_matrix(int(co[-1]), k, 40 + k)
        Y = host(B.spmm(dev(X)))
        for i, A in enumerate(mats):
            ref = oracle.csr_spmm(A, X[co[i]:co[i + 1]])
            s = oracle.csr_absmv(A, np.ascontiguousarray(X[co[i]:co[i + 1], k - 1]))
            assert oracle.scaled_error(np.ascontiguousarray(Y[ro[i]:ro[i + 1], k - 1]), ref[:, k - 1], s) <= TOL_F32
    A = W.zipf_matrix(6000, max_len=1500, seed=9)
    M = rg.rgcsr_from_csr(A, sigma=512, tau=12, col_panels=8)
    for k in (2, 3, 4, 5, 6, 8, 9, 12, 20):
        say("spmm panels", k)
        check(oracle, torch, A, M, k, np.float32)
        check(oracle, torch, A, M, k, np.float32, pad=1, off=1)
    bad = np.array([0, 17, A.n_cols - 1])
    X = W.uniform_matrix(A.n_cols, 6, 60)
    X[bad, 2] = [np.nan, np.inf, -np.inf]
    L = rg.rgcsr_from_csr(A, sigma=512, tau=12)
    Y = host(L.spmm(dev(X)))
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.row_ptr))
    hit = np.zeros(A.n_rows, bool)
    hit[rows[np.isin(A.col, bad)]] = True
    np.testing.assert_array_equal(np.isfinite(Y[:, 2]), ~hit)
    assert np.isfinite(np.delete(Y, 2, axis=1)).all()
