"""Max-convolution through the global buffer (4096 < n + m - 1 <= 16384) with
the family in several chunks: both transform lengths, pairs that are decided
in the first chunk next to pairs that need the smallest p, zero vectors, an
odd number of p, and p that are no powers of two.  Bar: the per-index FFT
bound of test_gpu_maxconv.py."""

import numpy as np
import pytest

import oracle
from test_gpu_maxconv import _dev, compare
from workloads import maxconv_vectors

pytestmark = pytest.mark.gpu


def _pairs(b, n, m, seed):
    """Kinds in turn, a pair of ones (every index decided at the largest p)
    and a pair with a zero vector."""
    kinds = ("uniform", "sparse", "lognormal", "distribution")
    x = np.empty((b, n))
    y = np.empty((b, m))
    for i, kind in enumerate(kinds):
        rows = len(range(i, b, 4))
        x[i::4], y[i::4] = maxconv_vectors(rows, n, m, seed + i, kind)
    x[1], y[1] = 1.0, 1.0
    if b > 2:
        y[b - 1] = 0.0
    return x, y


@pytest.mark.parametrize("b,n,m,P", [
    (80, 2100, 2003, [1, 2, 4, 8, 16, 32, 64]),           # 8192 points, chunks of 4 and 3
    (13, 8001, 300, list(range(1, 25))),                  # 16384 points, 24 p in chunks
    (45, 4000, 4500, [1, 3, 8, 20, 64, 100, 128]),        # 16384 points, p that are no powers of two
    (3, 8192, 8193, [2, 16, 64]),                         # the longest, one chunk
    (2, 4097, 1, [8]),                                    # the shortest, one p
], ids=["8192", "24p", "mixed", "longest", "shortest"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_chunks(gpu_lib, dtype, b, n, m, P):
    x, y = _pairs(b, n, m, 7)
    x, y = x.astype(dtype), y.astype(dtype)
    z, ps = gpu_lib.maxconv(_dev(x), _dev(y), P, return_pstar=True)
    compare(z.cpu().numpy(), ps.cpu().numpy(), x, y, P, oracle.TAU_FFT, fp32_out=dtype == np.float32)
