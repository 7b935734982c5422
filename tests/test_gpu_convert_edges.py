"""The device converter where its element-parallel kernels can go wrong: a
column out of order or out of range at any place of a four-element load, of a
row and of the array is refused (and a decrease across a row's border is not),
and long rows at the edges of the copied pieces arrive whole."""
import numpy as np
import pytest

from gpu_util import dev, say
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


def rows_of(lens, n_cols, seed=1):
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n_cols, l, replace=False)) for l in lens]
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate(cols).astype(np.int32) if cols else np.zeros(0, np.int32)
    return W.CSR(len(lens), n_cols, ptr, col, np.arange(1, len(col) + 1, dtype=np.float32))


def refused(A, rp, col):
    with pytest.raises(rg.RgcsrError) as e:
        rg.rgcsr_from_csr_device(A.n_rows, A.n_cols, dev(rp), dev(col), dev(A.val), rg.make_opts(G=64))
    return e.value.status, str(e.value)


@pytest.mark.parametrize("lens", [[9], [1, 0, 2, 0, 0, 5, 3], [4, 4, 4], [1030, 0, 3, 2500], [1] * 300 + [2]])
def test_order_and_range_at_every_place(torch_cuda, lens):
    A = rows_of(lens, 5000)
    say("converter order", lens[:8])
    on_device(torch_cuda, A, G=64)
    first = set(A.row_ptr[:-1].tolist())
    nnz = A.nnz
    places = range(nnz) if nnz <= 32 else sorted({0, 1, 3, 4, 5, 7, 8, 1023, 1024, 1025, 1026, nnz - 5, nnz - 2,
                                                  nnz - 1} & set(range(nnz)))
    for k in places:
        for bad in (-1, 5000):
            col = A.col.copy()
            col[k] = bad
            status, what = refused(A, A.row_ptr, col)
            assert status == 2 and "out of range" in what
        col = A.col.copy()
        if k in first:      # no smaller than the column before it, which is another row's
            if k and col[k - 1] < 4999 and (k + 1 in first or k + 1 == nnz):
                for c in (col[k - 1], col[k - 1] + 1, 0):
                    col[k] = c
                    on_device(torch_cuda, W.CSR(A.n_rows, A.n_cols, A.row_ptr, col, A.val), G=64)
        else:
            col[k] = col[k - 1]     # repeated
            assert "ascending" in refused(A, A.row_ptr, col)[1]
    rp = A.row_ptr.copy()
    rp[-1] -= 1
    assert refused(A, rp, A.col)[0] == 2


@pytest.mark.parametrize("lens", [[2047, 2048, 2049, 512, 511, 513, 30, 17, 3], [524288 + 2048 + 5, 4096, 20, 600000],
                                  [2049], [40] * 9 + [5000]])
def test_long_rows_in_pieces(torch_cuda, lens):
    A = rows_of(lens, 700000)
    say("converter long rows", lens[:6])
    for dt in ("f32", "bf16"):
        same_handles(on_device(torch_cuda, A, G=64, sigma=512, tau=16, value_dtype=dt),
                     rg.rgcsr_from_csr(A, G=64, sigma=512, tau=16, value_dtype=dt))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 9001, 1024 * 1025 + 7])
@pytest.mark.parametrize("sigma", [1, 2, 3, 512, 4095, 4096, 4097, 1 << 40])
def test_window_order_and_split(torch_cuda, n, sigma):
    """Many rows of equal length (the order within a length is the rows' own),
    windows on both sides of the largest that is sorted in LDS, and tiles of
    the split that hold only short rows, only long ones and none."""
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 5, n)
    lens[n // 3:n // 2] = 4
    cols = np.arange(lens.sum()) - np.repeat(np.concatenate([[0], np.cumsum(lens)[:-1]]), lens)
    A = W.CSR(n, 7, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), cols.astype(np.int32),
              np.arange(1, len(cols) + 1, dtype=np.float32))
    say("converter windows", n, sigma)
    for tau in (-1, 0, 2, 4):
        same_handles(on_device(torch_cuda, A, G=64, sigma=sigma, tau=tau), rg.rgcsr_from_csr(A, G=64, sigma=sigma, tau=tau))
