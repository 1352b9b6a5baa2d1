"""The one-kernel FP64 product at the edges of its split of the inner
dimension: 1, 2, 4, 8 and 16 waves of 32 inner indices, and rounds of 512
beyond, on tiles with one row or column more or less than 16, against the
oracle at the FP64 path's tolerance."""

import numpy as np
import pytest

import oracle
from parity import TAU, compare_estimate
from test_gpu_small_product import P64, _est, _launches
from workloads import lognormal_product, uniform_product

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 7, 8, 9, 31, 32, 33, 64, 65, 128, 129, 256, 257, 511, 512, 513, 1025, 1600])
@pytest.mark.parametrize("m,n", [(16, 16), (15, 33), (49, 17)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_inner_split(gpu_lib, m, n, k, dtype):
    draw = lognormal_product if k % 2 else uniform_product
    A, B = (x.astype(dtype) for x in draw(m, k, n, seed=31 * k + m))
    A[m // 2, :] = 0.0
    if k > 40:
        B[40:, 0] = 0.0
    assert _launches(gpu_lib, A, B, P64) == (1, 1)
    C, ps = _est(gpu_lib, A, B, P64)
    ref = oracle.pnorm_estimate(A, B, P64, TAU["fp64"])
    compare_estimate(C.astype(np.float64), ps, ref, P64, "fp64")
