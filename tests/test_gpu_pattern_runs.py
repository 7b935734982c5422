"""Row patterns whose x is copied to LDS in runs of nearby offsets: the same
bits as an explicit schedule over the layout's own columns, at the edges of
what makes a run (offsets 64 and 65 apart), of how many there are (3, 9, 10)
and of how far they reach, on matrices whose rows end inside a workgroup, with
runs that leave the matrix on both sides, empty rows and a strided x."""
import numpy as np
import pytest

from gpu_util import dev, host, say
from test_gpu_compact import both, diagonals

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


def box(runs, each, step=1):
    return [r + step * e for r in runs for e in range(-(each // 2), each - each // 2)]


OFFSETS = {
    "27 points": box([a * 900 + b * 30 for a in (-1, 0, 1) for b in (-1, 0, 1)], 3),
    "9 points": box([-70, 0, 70], 3),
    "gap 64": box([-66 * 2, -66, 0, 66, 66 * 2], 3),            # one run
    "gap 65": box([-67 * 2, -67, 0, 67, 67 * 2], 5, 1),         # gaps of 63
    "gaps of 65": list(range(0, 27 * 65, 65)),                  # 27 runs: gathered
    "nine runs": box(range(-400, 401, 100), 3),
    "ten runs": box(range(-400, 501, 100), 3),
    "wide runs": box([-1000, 0, 1000], 9, 10),                  # 240 entries behind the runs
    "too wide runs": box([-1000, 0, 1000], 9, 11),              # 264
    "25 points": box(range(-200, 201, 100), 5),
    "one side": list(range(0, 30)),
    "far out": box([-3000, 0, 3000], 9),
}


@pytest.mark.parametrize("vt", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("name", list(OFFSETS))
def test_runs(torch_cuda, oracle, name, vt):
    for n in (4096, 4096 + 255, 5121):
        A = diagonals(n, n, OFFSETS[name], dtype=np.float64 if vt == "f64" else np.float32)
        say("pattern runs", name, vt, n)
        assert both(oracle, torch_cuda, A, vt) > 0
    A = diagonals(4999, 6001, OFFSETS[name], dtype=np.float64 if vt == "f64" else np.float32, drop=0.3)
    both(oracle, torch_cuda, A, vt)
    if vt == "f32":
        both(oracle, torch_cuda, A, vt, vec=np.float64)
        both(oracle, torch_cuda, A, vt, sort=64)    # rows out of order: gathered
        both(oracle, torch_cuda, A, vt, G=128)


@pytest.mark.parametrize("vt,vec", [("f32", np.float32), ("f64", np.float64)])
def test_runs_of_a_strided_x(torch_cuda, oracle, vt, vec):
    torch = torch_cuda
    A = diagonals(5121, 5121, OFFSETS["27 points"], dtype=vec)
    M = rg.rgcsr_from_csr(A, value_dtype=vt)
    x = dev(W.uniform_vector(A.n_cols, 3, vec))
    X = torch.full((A.n_cols, 3), 5.0, dtype=x.dtype, device="cuda:0")
    X[:, 0] = x
    Y = torch.full((A.n_rows, 2), 7.0, dtype=x.dtype, device="cuda:0")
    say("pattern runs strided", vt)
    _lib.call("rgcsr_spmv_batched", M.handle, 1, X.data_ptr(), 3, Y.data_ptr(), 2, rg._code_of_tensor(x), 0,
              torch.cuda.current_stream().cuda_stream)
    Yh, y = host(Y), host(M.spmv(x))
    np.testing.assert_array_equal(np.ascontiguousarray(Yh[:, 0]).view(np.uint8), y.view(np.uint8))
    assert np.all(Yh[:, 1] == 7.0)
