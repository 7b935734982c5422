"""GPU test of one right-hand side into a strided Y (k = 1, ldx = 1, ldy > 1)
on handles whose SpMV takes the two steps: every kind of row it multiplies,
against the same product into a contiguous y."""
import numpy as np
import pytest

from gpu_util import dev, host, say

import paper_1012_2270_amd as rg
from paper_1012_2270_amd import _lib
from paper_1012_2270_amd import workloads as W
from test_gpu_expand import LONGS, skewed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ldy", [2, 3])
@pytest.mark.parametrize("vt", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("lay", [dict(sigma=512, tau=6), dict(tau=16)])
def test_strided_y(lay, vt, ldy):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # row groups (some rows empty), wavefront rows, rows of one chunk, and one
    # of two chunks, whose sums a kernel of their own adds
    # (FP64 takes the two steps at larger sizes)
    big = vt == "f64"
    A = skewed(200_037 if big else 40_037, 400_001 if big else 50_001, 1,
               LONGS * (4 if big else 1) + [16_384 + 4096 + 5], empty=0.03)
    M = rg.rgcsr_from_csr(A, value_dtype=vt, **lay)
    # the same rows in column tiles take other memory: M does not hold tiles
    T = rg.rgcsr_from_csr(A, value_dtype=vt, tile_min_len=256, **lay)
    assert M.info["tiled_rows"] == T.info["tiled_rows"] > 0 and M.info["device_bytes"] != T.info["device_bytes"]
    x = dev(W.uniform_vector(A.n_cols, 2, np.float64 if vt == "f64" else np.float32))
    Y = torch.full((A.n_rows, ldy), 7.0, dtype=x.dtype, device="cuda:0")
    say("two-step, strided y", vt, ldy, lay)
    _lib.call("rgcsr_spmv_batched", M.handle, 1, x.data_ptr(), 1, Y.data_ptr(), ldy, rg._code_of_tensor(x), 0,
              torch.cuda.current_stream().cuda_stream)
    got, y = host(Y), host(M.spmv(x))
    np.testing.assert_array_equal(np.ascontiguousarray(got[:, 0]).view(np.uint8), y.view(np.uint8))
    assert np.all(got[:, 1:] == 7.0)
