"""The automatic column tiles that a handle in caller memory keeps, where one
that owns its memory takes the two-step SpMV: the same bits as tiles asked for
by length, at full size."""
import numpy as np
import pytest

from gpu_util import TOL_F32, TOL_F64, check_spmv, dev, host, say

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


@pytest.mark.parametrize("vt", ["f32", "f64"])
def test_automatic_tiles_in_caller_memory(torch_cuda, oracle, vt):
    """The benchmark's Zipf matrix in a plan: tiles chosen by themselves."""
    A, x = W.workload_zipf()
    if vt == "f64":
        A, x = W.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col, A.val.astype(np.float64)), x.astype(np.float64)
    lay = dict(sigma=512, tau=6)
    say("automatic tiles in caller memory", vt)
    M = rg.rgcsr_plan_from_csr(A, value_dtype=vt, **lay).build()
    T = rg.rgcsr_from_csr(A, value_dtype=vt, tile_min_len=256, **lay)
    assert M.info["tiled_rows"] == T.info["tiled_rows"] > 1000
    assert M.info["device_bytes"] <= T.info["device_bytes"]  # no other form beside the tiles
    y = host(M.spmv(dev(x)))
    check_spmv(oracle, A, x, y, tol=TOL_F64 if vt == "f64" else TOL_F32)
    np.testing.assert_array_equal(host(T.spmv(dev(x))).view(np.uint8), y.view(np.uint8))
