"""Row patterns and x windows found on the host: a row that differs from the one
before it in one column, in its length or in nothing, at the edges of a group
and of a row, in the rows' own order, sorted and in a batch, gives the same
bits as an explicit schedule and as the search on the device."""
import numpy as np
import pytest

from gpu_util import dev, host, say
from test_gpu_compact import both, diagonals

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


@pytest.mark.parametrize("sort", [1, 64])
@pytest.mark.parametrize("row", [640, 641, 670, 703])
def test_one_row_differs(torch_cuda, oracle, row, sort):
    A = diagonals(2048, 2048, np.array([-9, -4, 0, 3, 8]))
    b = A.row_ptr[row]
    for j in range(5):
        col = A.col.copy()
        col[b + j] += 1
        say("one column", row, j, sort)
        assert both(oracle, torch_cuda, W.CSR(2048, 2048, A.row_ptr, col, A.val), "f32", sort=sort) > 0
    keep = np.ones(A.nnz, bool)
    keep[b + 4] = False
    rp = A.row_ptr - (np.arange(2049) > row)
    say("one entry less", row, sort)
    assert both(oracle, torch_cuda, W.CSR(2048, 2048, rp, A.col[keep], A.val[keep]), "f32", sort=sort) > 0
    keep[b:b + 5] = False
    say("no entries", row, sort)
    assert both(oracle, torch_cuda, W.CSR(2048, 2048, A.row_ptr - 5 * (np.arange(2049) > row), A.col[keep], A.val[keep]),
                "f32", sort=sort) > 0


def banded(n, seed):
    """Rows of 6 to 24 columns in a band of 400, some and a whole group's empty."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(6, 25, n)
    lens[::50] = 0
    lens[128:192] = 0
    lo = np.maximum(np.arange(n) - 200, 0)
    hi = np.minimum(np.arange(n) + 200, n)
    col = W._unique_sorted_columns(rng, lens, lo, hi)
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    return W.CSR(n, n, rp, col, rng.standard_normal(int(rp[-1])).astype(np.float32))


@pytest.mark.parametrize("sort", [1, 256])
def test_windows(torch_cuda, oracle, sort):
    A = banded(20_003, 5)
    say("windows", sort)
    assert both(oracle, torch_cuda, A, "f32", sort=sort) > 2 * A.nnz


@pytest.mark.parametrize("kind", ["patterns", "windows"])
def test_batch(torch_cuda, oracle, kind):
    mats = [diagonals(700 + 65 * i, 700 + 65 * i, np.array([-9, -4, 0, 3, 8])) if kind == "patterns" else banded(5000 + 65 * i, i)
            for i in range(5)]
    M, E = rg.rgcsr_from_csr_batch(mats), rg.rgcsr_from_csr_batch(mats, pad_loads=0)
    assert M.info["device_bytes"] > E.info["device_bytes"]
    x = dev(W.uniform_vector(sum(A.n_cols for A in mats), 3, np.float32))
    say("batch", kind)
    np.testing.assert_array_equal(host(M.spmv(x)).view(np.uint32), host(E.spmv(x)).view(np.uint32))
