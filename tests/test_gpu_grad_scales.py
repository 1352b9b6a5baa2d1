"""The backward's power planes scale by plane column (c of B, r of A): whole
and ragged chunks of 8, zero lines, lines whose scale has no normal
reciprocal, against the oracle's gradient at the tolerance of
test_gpu_grad.py (the quotient from a reciprocal and its remainder is the
division's up to its last bit)."""

import numpy as np
import pytest

import oracle
from parity import TAU
from test_gpu_grad import TOL, _check, _gpu_grad
from workloads import gradient_case

pytestmark = pytest.mark.gpu

P = [1, 2, 4, 8, 16, 32, 64]


@pytest.mark.parametrize("m,k,n", [(72, 64, 264), (70, 64, 261), (65, 33, 8), (300, 40, 63)])
@pytest.mark.parametrize("path", ["fp64", "bf16"])
def test_column_scales(gpu_lib, m, k, n, path):
    dt = np.float64 if path == "fp64" else np.float32
    A, B, G = (x[0] for x in gradient_case(1, m, k, n, seed=m + n, dtype=dt))
    A[3] = 0.0
    B[:, n // 2] = 0.0
    A[9] *= dt(1e-310 if path == "fp64" else 1e-30)  # no normal reciprocal / a large one
    B[:, 2] *= dt(1e-200 if path == "fp64" else 1e-20)
    A[11] *= dt(1e+200 if path == "fp64" else 1e+3)
    G[11] *= dt(1e-200 if path == "fp64" else 1e-3)
    _, ps, dA, dB = _gpu_grad(gpu_lib, A, B, G, P, path)
    rA, rB = oracle.pnorm_grad(A, B, G, P, ps)
    assert np.isfinite(dA).all() and np.isfinite(dB).all()
    _check(dA, rA, TOL[path])
    _check(dB, rB, TOL[path])
