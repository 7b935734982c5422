"""SpMM over handles on both sides of the padding and of the row count from
which X rows past a row's length are left out, and of those where four FP64
columns take one lane per row: every column the bits of a single-column launch
where no row is long, against the oracle where some are."""
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


def rows_of(n, kind, dtype):
    """Equal rows of 12 (no padding), rows of 0 to 8 (padding as large as the
    nonzeros, empty rows), or those with some long ones."""
    rng = np.random.default_rng(n)
    lens = np.full(n, 12, np.int64) if kind == "equal" else rng.integers(0, 9, n)
    if kind == "long":
        lens[rng.choice(n, 40, replace=False)] = 700
        lens[n // 2] = 18_000
    col = W._unique_sorted_columns(rng, lens, np.zeros(n, np.int64), np.full(n, 30_000, np.int64))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    return W.CSR(n, 30_000, rp, col, rng.standard_normal(int(rp[-1])).astype(dtype))


@pytest.mark.parametrize("vt,vec", [("f32", np.float32), ("f64", np.float64), ("f32", np.float64)])
@pytest.mark.parametrize("kind,n", [("equal", 2048 * 64), ("short", 2048 * 64 - 1), ("short", 2048 * 64),
                                    ("long", 1024 * 64 - 1), ("long", 1024 * 64 + 41)])  # 41 long rows
def test_padding(torch_cuda, oracle, n, kind, vt, vec):
    A = rows_of(n, kind, np.float64 if vt == "f64" else np.float32)
    M = rg.rgcsr_from_csr(A, value_dtype=vt, **(dict(tau=10) if kind == "long" else {}))
    for k in (3, 4, 7, 8, 16, 17, 32):
        say("spmm padding", n, kind, vt, vec.__name__, k)
        check(oracle, torch_cuda, A, M, k, vec, pad=k % 2, bits=kind != "long")


def test_non_finite_x(torch_cuda, oracle):
    """Rows that do not use a non-finite entry stay finite."""
    torch = torch_cuda
    A = rows_of(2048 * 64, "short", np.float32)
    X = W.uniform_matrix(A.n_cols, 8, 3, np.float32)
    bad = np.array([0, 77, 29_999])
    X[bad] = np.array([np.nan, np.inf, -np.inf])[:, None]
    say("spmm padding, non-finite X")
    Y = rg.rgcsr_from_csr(A).spmm(torch.from_numpy(X).cuda()).cpu().numpy()
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.row_ptr))
    hit = np.zeros(A.n_rows, bool)
    hit[rows[np.isin(A.col, bad)]] = True
    np.testing.assert_array_equal(np.isfinite(Y), np.repeat(~hit[:, None], 8, 1))
