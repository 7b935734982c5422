"""Row patterns on both sides of the widths and run counts from which x is
copied to LDS in runs rather than gathered: the same bits as an explicit
schedule over the layout's own columns."""
import numpy as np
import pytest

from gpu_util import say
from test_gpu_compact import both, diagonals

import paper_1012_2270_amd as rg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg._lib.load()
    return torch


# runs x offsets of each: 7 and 8 wide, 15 and 16, 17 and 18, in 1 to 9 runs
@pytest.mark.parametrize("vt,vec", [("f64", np.float64), ("f32", np.float64), ("f32", np.float32)])
@pytest.mark.parametrize("runs,each", [(1, 7), (1, 8), (2, 4), (3, 3), (3, 5), (1, 16), (2, 8), (4, 2), (4, 4), (1, 17),
                                       (6, 3), (9, 2), (5, 5), (9, 3)])
def test_edges(torch_cuda, oracle, runs, each, vt, vec):
    offs = [200 * (r - runs // 2) + e for r in range(runs) for e in range(each)]
    say("run rules", runs, each, vt, vec.__name__)
    for n in (2048, 3333):
        A = diagonals(n, n, offs, dtype=np.float64 if vt == "f64" else np.float32)
        assert both(oracle, torch_cuda, A, vt, vec=vec) > 0
