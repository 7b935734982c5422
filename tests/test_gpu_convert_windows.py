"""The window order of the device converter with windows that share a
workgroup: windows around its 128 rows, and as many rows in windows of two as
a workgroup per window could not be launched for (2^26 of 64 threads)."""
import numpy as np
import pytest

from gpu_util import say
from test_gpu_convert import on_device, same_handles

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


@pytest.mark.parametrize("n", [127, 128, 129, 4097])
@pytest.mark.parametrize("sigma", [2, 3, 5, 31, 42, 43, 63, 64, 65, 127, 128, 129])
def test_windows_that_share_a_workgroup(torch_cuda, n, sigma):
    rng = np.random.default_rng(n + sigma)
    lens = rng.integers(0, 5, n)
    lens[n // 3:n // 2] = 4
    cols = np.arange(lens.sum()) - np.repeat(np.concatenate([[0], np.cumsum(lens)[:-1]]), lens)
    A = W.CSR(n, 7, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), cols.astype(np.int32),
              np.arange(1, len(cols) + 1, dtype=np.float32))
    say("converter windows", n, sigma)
    for tau in (-1, 2):
        same_handles(on_device(torch_cuda, A, G=64, sigma=sigma, tau=tau), rg.rgcsr_from_csr(A, G=64, sigma=sigma, tau=tau))


def test_many_rows_in_windows_of_two(torch_cuda):
    torch = torch_cuda
    n = 1 << 27
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1)
    rows = torch.unique(torch.randint(n, (50_000,), generator=g, device="cuda:0"))
    rows[-1] = n - 1
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
    rp[rows + 1] = 1
    rp = rp.cumsum(0)
    col = torch.randint(1000, (rows.numel(),), generator=g, device="cuda:0", dtype=torch.int32)
    val = torch.rand(rows.numel(), generator=g, device="cuda:0")
    x = torch.rand(1000, generator=g, device="cuda:0")
    say("converter, 2^27 rows in windows of two")
    M = rg.rgcsr_from_csr_device(n, 1000, rp, col, val, rg.make_opts(G=64, sigma=2))
    y = M.spmv(x)
    # a row holds one product or nothing: the same bits
    assert torch.equal(y[rows], val * x[col.long()])
    y[rows] = 0
    assert int(torch.count_nonzero(y)) == 0
    M.close()
