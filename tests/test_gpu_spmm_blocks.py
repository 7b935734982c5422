"""More right-hand sides than one launch takes: the blocks of columns that a
call runs, at the edges of their widths, and 33 columns of more than 4 GiB,
which no single-column launch may be left of."""
import numpy as np
import pytest

from gpu_util import say

import paper_1012_2270_amd as rg
from paper_1012_2270_amd import workloads as W
from test_gpu_spmm_widths import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg._lib.load()
    return torch


@pytest.mark.parametrize("vt,vec", [("f32", np.float32), ("f64", np.float64)])
@pytest.mark.parametrize("k", [33, 34, 36, 48, 63, 64, 65, 66, 97])
def test_blocks(torch_cuda, oracle, k, vt, vec):
    A = W.random_csr(900, 40_000, seed=4, max_len=200, long_rows=6, long_len=20_000).astype(vec)
    S = W.random_csr(2500, 1900, seed=3, max_len=14, empty_frac=0.2).astype(vec)
    M, MS = rg.rgcsr_from_csr(A, value_dtype=vt, sigma=64, tau=10), rg.rgcsr_from_csr(S, value_dtype=vt, sigma=300)
    say("spmm blocks", k, vt)
    check(oracle, torch_cuda, A, M, k, vec, pad=1)
    check(oracle, torch_cuda, S, MS, k, vec, bits=True)


def test_33_columns_of_more_than_4_gib(torch_cuda):
    torch = torch_cuda
    n, k = 1 << 25, 33
    col = np.linspace(0, n - 1, 700).astype(np.int32)
    A = W.CSR(100, n, np.arange(0, 701, 7, dtype=np.int64), col, np.arange(1, 701, dtype=np.float32))
    M = rg.rgcsr_from_csr(A)
    X = torch.rand(n, k, device="cuda:0")
    assert X.numel() * 4 >= 1 << 32
    say("spmm, 33 columns of more than 4 GiB")
    Y = M.spmm(X)
    ref = (torch.from_numpy(A.val).double()[:, None].cuda() * X[torch.from_numpy(col).long().cuda()].double())
    ref = ref.reshape(100, 7, k).sum(1)
    # sums of seven FP32 products
    assert float(((Y.double() - ref).abs() / ref).max()) <= 8 * 2.0 ** -24
