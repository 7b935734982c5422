"""Conjugate gradients at the sizes where the vector kernels can go wrong:
one workgroup and its edges, the vector's ragged end, more rows than one pass
of 256 workgroups, and vectors that start at an odd element.  The matrix is
tridiagonal, 3 on the diagonal and -1 beside it (condition at most 5), so a
residual of 1e-10 takes some 30 iterations and the recurrence's residual
differs from the true one by about 5 * 30 * 2^-53, far below 1% of 1e-10."""
import math

import numpy as np
import pytest

from gpu_util import dev, host, say

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


def tridiagonal(n):
    i = np.repeat(np.arange(n), 3)
    c = i + np.tile([-1, 0, 1], n)
    v = np.tile([-1.0, 3.0, -1.0], n)
    keep = (c >= 0) & (c < n)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(i[keep], minlength=n))])
    return W.CSR(n, n, ptr.astype(np.int64), c[keep].astype(np.int32), v[keep])


@pytest.mark.parametrize("n", [61, 4095, 4096, 4097, 8195, 4096 * 255 + 2, 4096 * 256, 2100003])
def test_cg_sizes(torch_cuda, oracle, n):
    torch = torch_cuda
    A = tridiagonal(n)
    xs = W.uniform_vector(n, 7)
    b = oracle.csr_spmv(A, xs)
    bnorm = math.sqrt(float(np.dot(b, b)))
    M = rg.rgcsr_from_csr(A, value_dtype="f64")
    lo = rg.rgcsr_from_csr(A, value_dtype="bf16")
    off = torch.zeros(n + 1, dtype=torch.float64, device="cuda:0")
    off[1:] = dev(b)
    bd = off[1:]
    _, it_orc, _ = oracle.cg(A, b, tol=1e-10)
    say("cg sizes", n, "oracle iterations", it_orc)
    xd = torch.zeros(n + 1, dtype=torch.float64, device="cuda:0")
    st = rg.rgcsr_cg_solve_f64(M, bd, xd[1:], tol=1e-10)
    r = b - oracle.csr_spmv(A, host(xd)[1:])
    assert math.sqrt(float(np.dot(r, r))) / bnorm <= 1.01e-10
    assert abs(st["inner_iterations"] - it_orc) <= 4
    assert float(xd[0].item()) == 0.0
    # iterations that end between two checks
    xm = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    assert rg.rgcsr_cg_solve_f64(M, bd, xm, tol=1e-10, max_iter=6)["inner_iterations"] == 6
    runs = []
    for solve in (rg.rgcsr_cg_solve, rg.rgcsr_cg_solve) + ((rg.rgcsr_cg_solve_noalloc,) if n <= 1 << 20 else ()):
        xd = torch.zeros(n + 1, dtype=torch.float64, device="cuda:0")
        st = solve(lo, M, bd, xd[1:], tol=1e-10, inner_tol=1e-4)
        xh = host(xd)
        r = b - oracle.csr_spmv(A, xh[1:])
        assert st["converged"] and math.sqrt(float(np.dot(r, r))) / bnorm <= 1.01e-10
        runs.append((xh.tobytes(), st["outer_iterations"], st["inner_iterations"], st["relres"]))
    assert all(t == runs[0] for t in runs)   # the same bits every time, with either workspace
    assert rg.rgcsr_cg_solve(lo, M, bd, torch.zeros(n, dtype=torch.float64, device="cuda:0"), max_outer=1,
                             max_inner=5)["inner_iterations"] == 5


@pytest.mark.parametrize("n", [61, 4097, 40001])
@pytest.mark.parametrize("G", [64, 128, 32])
def test_cg_product_and_its_sum(torch_cuda, oracle, n, G):
    """p.q from the SpMV (row patterns: whole wavefronts of rows) and from a
    kernel of its own (G = 32): the same solution, iterations within one check
    of the oracle's."""
    torch = torch_cuda
    A = tridiagonal(n)
    b = oracle.csr_spmv(A, W.uniform_vector(n, 8))
    M = rg.rgcsr_from_csr(A, value_dtype="f64", G=G)
    lo = rg.rgcsr_from_csr(A, value_dtype="f32", G=G)
    _, it_orc, _ = oracle.cg(A, b, tol=1e-10)
    say("cg sum", n, G)
    for solve in (lambda x: rg.rgcsr_cg_solve_f64(M, dev(b), x, tol=1e-10), lambda x: rg.rgcsr_cg_solve(lo, M, dev(b), x)):
        xd = torch.zeros(n, dtype=torch.float64, device="cuda:0")
        st = solve(xd)
        r = b - oracle.csr_spmv(A, host(xd))
        assert math.sqrt(float(np.dot(r, r)) / float(np.dot(b, b))) <= 1.01e-10
        if st["outer_iterations"] == 0:
            assert abs(st["inner_iterations"] - it_orc) <= 4
