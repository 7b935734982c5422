"""The two-step SpMV in FP64 storage, which takes more nonzeros than in the
other types, on both sides of that line (below it: the same bits as column
tiles asked for by length)."""
import numpy as np
import pytest

from gpu_util import TOL_F64, check_spmv, dev, host, say

import paper_1012_2270_amd as rg
from paper_1012_2270_amd import workloads as W
from test_gpu_expand import LONGS, skewed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg._lib.load()
    return torch


@pytest.mark.parametrize("lay", [dict(sigma=512, tau=6), dict(tau=16)])
@pytest.mark.parametrize("n_cols,copies,two_steps", [(50_001, 5, True), (400_001, 5, True), (400_001, 3, False)])
def test_parity(torch_cuda, oracle, n_cols, copies, two_steps, lay):
    A = skewed(150_037, n_cols, 1, LONGS * copies + [16_384 + 4096 + 5], empty=0.03, dtype=np.float64)
    assert (A.nnz >= 2_200_000) == two_steps
    x = dev(W.uniform_vector(n_cols, 2, np.float64))
    say("two-step FP64", n_cols, A.nnz, lay)
    M = rg.rgcsr_from_csr(A, value_dtype="f64", **lay)
    T = rg.rgcsr_from_csr(A, value_dtype="f64", tile_min_len=256, **lay)
    assert M.info["tiled_rows"] == T.info["tiled_rows"] > 0
    assert (M.info["device_bytes"] != T.info["device_bytes"]) == two_steps
    y = host(M.spmv(x))
    check_spmv(oracle, A, host(x), y, tol=TOL_F64)
    np.testing.assert_array_equal(host(M.spmv(x)).view(np.uint64), y.view(np.uint64))
    D = rg.rgcsr_from_csr_device(A.n_rows, A.n_cols, dev(A.row_ptr), dev(A.col), dev(A.val),
                                 rg.make_opts(value_dtype="f64", **lay))
    np.testing.assert_array_equal(host(D.spmv(x)).view(np.uint64), y.view(np.uint64))
    if not two_steps:
        np.testing.assert_array_equal(host(T.spmv(x)).view(np.uint64), y.view(np.uint64))
