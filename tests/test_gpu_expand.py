"""GPU tests of the two-step SpMV (x expanded through LDS tiles, then
multiplied unit by unit) against the oracle, at the edges of its tiles, units
and runs.  It serves automatic column tiles on handles that own their memory."""
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


def skewed(n_rows, n_cols, seed, longs, short=5, empty=0.0, dtype=np.float32):
    """Rows of 0 to 2 * short nonzeros, the rows `longs` (position, length) long."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 2 * short + 1, n_rows)
    lens[rng.random(n_rows) < empty] = 0
    at = rng.choice(n_rows, len(longs), replace=False)
    lens[at] = longs
    lens = np.minimum(lens, n_cols)
    col = W._unique_sorted_columns(rng, lens, np.zeros(n_rows, np.int64), np.full(n_rows, n_cols, np.int64))
    rp = np.zeros(n_rows + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    return W.CSR(n_rows, n_cols, rp, col, rng.standard_normal(int(rp[-1])).astype(dtype))


def expanded(M, E):
    """The runs take 4 bytes and a vector element per entry, and rounding up."""
    return M.info["device_bytes"] - E.info["device_bytes"] > 8 * M.nnz


LONGS = [300] * 1000 + [1023, 1024, 1025, 4096, 4097, 9000]


# columns at the edges of the tiles (16,384 columns; 8,192 in FP64)
@pytest.mark.parametrize("vt", ["f32", "f64", "f16"])
@pytest.mark.parametrize("n_cols", [9000, 16383, 16384, 16385, 50_001])
@pytest.mark.parametrize("lay", [dict(sigma=512, tau=6), dict(tau=16), dict(sigma=256, tau=30)])
def test_parity(torch_cuda, oracle, n_cols, vt, lay):
    A = skewed(40_037, n_cols, 1, [l for l in LONGS if l < n_cols] + [16_384 + 4096 + 5] * (n_cols > 30_000),
               empty=0.03)
    vec = np.float64 if vt == "f64" else np.float32
    x = W.uniform_vector(n_cols, 2, vec)
    say("two-step", n_cols, vt, lay)
    M = rg.rgcsr_from_csr(A, value_dtype=vt, **lay)
    E = rg.rgcsr_from_csr(A, value_dtype=vt, tile_min_len=0, **lay)
    assert M.info["tiled_rows"] > 0 and expanded(M, E)
    xd = dev(x)
    y = host(M.spmv(xd))
    check_spmv(oracle, A, x, y, vals64=storage_values(oracle, A, vt), tol=TOL_F64 if vt == "f64" else TOL_F32)
    bits = np.uint64 if vt == "f64" else np.uint32
    np.testing.assert_array_equal(host(M.spmv(xd)).view(bits), y.view(bits))  # the same bits again
    D = rg.rgcsr_from_csr_device(A.n_rows, A.n_cols, dev(A.row_ptr), dev(A.col), dev(A.val),
                                 rg.make_opts(value_dtype=vt, **lay))
    assert D.info["tiled_rows"] == M.info["tiled_rows"]
    np.testing.assert_array_equal(host(D.spmv(xd)).view(bits), y.view(bits))


def test_unaligned_x_clone_and_other_vectors(torch_cuda, oracle):
    torch = torch_cuda
    A = skewed(30_000, 40_000, 3, LONGS)
    x = W.uniform_vector(A.n_cols, 4, np.float32)
    M = rg.rgcsr_from_csr(A, tau=16, sigma=512)
    y = host(M.spmv(dev(x)))
    buf = torch.empty(A.n_cols + 1, device="cuda:0")
    buf[1:] = dev(x)
    say("two-step, x at a 4-byte offset, clone, FP64 vectors, two columns")
    np.testing.assert_array_equal(host(M.spmv(buf[1:])).view(np.uint32), y.view(np.uint32))
    C = M.clone()
    M.close()
    np.testing.assert_array_equal(host(C.spmv(dev(x))).view(np.uint32), y.view(np.uint32))
    check_spmv(oracle, A, x, host(C.spmv(dev(x.astype(np.float64)))), tol=TOL_F32)
    X = W.uniform_matrix(A.n_cols, 2, 5)
    Y = host(C.spmm(dev(X)))
    for k in range(2):
        check_spmv(oracle, A, X[:, k].copy(), np.ascontiguousarray(Y[:, k]))


def test_value_update_transpose_and_backward(torch_cuda, oracle):
    torch = torch_cuda
    A = skewed(30_000, 30_000, 6, LONGS)
    x = W.uniform_vector(A.n_cols, 7, np.float32)
    theta = W.normal_vector(A.nnz, 8, np.float32)
    B = W.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col, theta)
    M = rg.rgcsr_from_csr(A, tau=16, sigma=512, build_transpose=True)
    say("two-step, value update and backward")
    rg.rgcsr_set_values(M, dev(theta))
    check_spmv(oracle, B, x, host(M.spmv(dev(x))))
    dy = W.normal_vector(A.n_rows, 9, np.float32)
    dx, dv = torch.empty(A.n_cols, device="cuda:0"), torch.empty(A.nnz, device="cuda:0")
    rg.rgcsr_spmv_transpose_grad(M, dev(x), dev(dy), dx, dv)
    T = W.CSR(A.n_cols, A.n_rows, *oracle.csr_transpose(B))
    check_spmv(oracle, T, dy, host(dx))
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.row_ptr))
    np.testing.assert_array_equal(host(dv).view(np.uint32), (dy[rows] * x[A.col]).view(np.uint32))
    # the transpose has the long rows when the columns are the crowded ones
    M2 = rg.rgcsr_from_csr(T, tau=16, sigma=512, build_transpose=True)
    rg.rgcsr_spmv_transpose_grad(M2, None, dev(x), dx, None)
    check_spmv(oracle, B, x, host(dx))


def test_batch_and_graph_replay(torch_cuda, oracle):
    torch = torch_cuda
    mats = [skewed(5000 + 700 * i, 9000 + 3000 * i, 10 + i, [400] * 350 + [5000], empty=0.05) for i in range(4)]
    B = rg.rgcsr_from_csr_batch(mats, tau=16, sigma=256)
    E = rg.rgcsr_from_csr_batch(mats, tau=16, sigma=256, tile_min_len=0)
    assert expanded(B, E)
    ro, co = B.batch_offsets()
    x = dev(W.uniform_vector(int(co[-1]), 20, np.float32))
    y = torch.empty(int(ro[-1]), device="cuda:0")
    say("two-step, batch and graph")
    rg.rgcsr_spmv(B, x, y)
    first = host(y).copy()
    for i, A in enumerate(mats):
        check_spmv(oracle, A, host(x)[co[i]:co[i + 1]], first[ro[i]:ro[i + 1]])
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        rg.rgcsr_spmv(B, x, y)
    torch.cuda.current_stream().wait_stream(s)
    with torch.cuda.graph(g):
        rg.rgcsr_spmv(B, x, y)
    for k in range(4):
        x.copy_(dev(W.uniform_vector(int(co[-1]), 21 + k, np.float32)))
        y.fill_(7.0)
        g.replay()
        got = host(y).copy()
        rg.rgcsr_spmv(B, x, y)  # eager work between the replays
        np.testing.assert_array_equal(got.view(np.uint32), host(y).view(np.uint32))


def test_non_finite_x(torch_cuda, oracle):
    A = skewed(20_000, 33_000, 30, LONGS, empty=0.1)
    x = W.uniform_vector(A.n_cols, 31, np.float32)
    bad = np.array([0, 16_383, 16_384, 32_999])
    x[bad] = [np.nan, np.inf, -np.inf, np.nan]
    say("two-step, non-finite x")
    y = host(rg.rgcsr_from_csr(A, tau=16, sigma=512).spmv(dev(x)))
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.row_ptr))
    hit = np.zeros(A.n_rows, bool)
    hit[rows[np.isin(A.col, bad)]] = True
    np.testing.assert_array_equal(np.isfinite(y), ~hit)
