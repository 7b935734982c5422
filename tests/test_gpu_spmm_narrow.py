"""SpMM of 2 and 4 columns over row patterns, on both sides of the row count and
width up to which one lane takes a row: the bits of single-column launches."""
import numpy as np
import pytest

from gpu_util import say
from test_gpu_compact import diagonals
from test_gpu_spmm_widths import check

import paper_1012_2270_amd as rg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg._lib.load()
    return torch


@pytest.mark.parametrize("vt,vec", [("f32", np.float32), ("f64", np.float64), ("f32", np.float64)])
@pytest.mark.parametrize("width", [5, 8, 9, 27])
@pytest.mark.parametrize("n", [300, 65_535, 65_536, 131_071, 131_072])
def test_patterns(torch_cuda, oracle, n, width, vt, vec):
    A = diagonals(n, n, np.arange(width) * 11 - 5 * width, dtype=np.float64 if vt == "f64" else np.float32)
    M = rg.rgcsr_from_csr(A, value_dtype=vt)
    for k in (2, 4):
        say("spmm patterns", n, width, vt, vec.__name__, k)
        check(oracle, torch_cuda, A, M, k, vec, bits=True)
