"""The backward where C overflows its type in one entry (documented where r c
S^(1/p) does) or a cotangent is infinite.  An infinite C has C'^(1-p) = 0 for
p > 1 and adds nothing, whatever its cotangent; an infinite cotangent reaches
its own row of dA and column of dB only, as that infinity.  The other lines
are the oracle's at the tolerance of test_gpu_grad.py."""

import numpy as np
import pytest

import oracle
from test_gpu_grad import TOL, _check, _gpu_grad
from workloads import gradient_case

pytestmark = pytest.mark.gpu

I0, J0 = 11, 29


def _lines(dA, dB, rA, rB, tol, skip=False):
    def check(got, ref):
        # (both in units of the largest entry: the norm of 1e200 overflows)
        unit = np.abs(ref).max()
        _check(got / unit, ref / unit, tol)

    if not skip:
        check(dA[I0], rA[I0])
        check(dB[:, J0], rB[:, J0])
    check(np.delete(dA, I0, 0), np.delete(rA, I0, 0))
    check(np.delete(dB, J0, 1), np.delete(rB, J0, 1))


@pytest.mark.parametrize("shape", [(64, 64, 64), (70, 45, 83)])
@pytest.mark.parametrize("P", [[2], [64], [1, 2, 4, 8, 16]], ids=str)
@pytest.mark.parametrize("cotangent", ["drawn", "zero"])
@pytest.mark.parametrize("path,dtype", [("fp64", np.float64), ("fp64", np.float32), ("bf16", np.float32)])
def test_overflowed_entry(gpu_lib, path, dtype, cotangent, P, shape):
    m, k, n = shape
    A, B, G = (x[0] for x in gradient_case(1, m, k, n, seed=m + n, dtype=dtype))
    big = dtype(1e25 if dtype == np.float32 else 1e200)
    A[I0] *= big
    B[:, J0] *= big
    if cotangent == "zero":
        G[I0, J0] = 0
    print(f"[grad inf] C {path} {dtype.__name__} {shape} {P} {cotangent}", flush=True)
    C, ps, dA, dB = _gpu_grad(gpu_lib, A, B, G, P, path)
    assert np.isinf(C[I0, J0]) and np.isfinite(np.delete(C.ravel(), I0 * n + J0)).all()
    G0 = G.copy()
    G0[I0, J0] = 0
    rA, rB = oracle.pnorm_grad(A, B, G0, P, ps)
    _lines(dA, dB, rA, rB, TOL[path])


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("P", [[1], [2], [1, 2, 4, 8, 16]], ids=str)
def test_infinite_cotangent(gpu_lib, P, sign):
    A, B, G = (x[0] for x in gradient_case(1, 70, 45, 83, seed=5, dtype=np.float64))
    G0 = G.copy()
    G0[I0, J0] = 0
    G[I0, J0] = sign * np.inf
    print(f"[grad inf] G {P} {sign}", flush=True)
    _, ps, dA, dB = _gpu_grad(gpu_lib, A, B, G, P, "fp64")
    rA, rB = oracle.pnorm_grad(A, B, G0, P, ps)
    _lines(dA, dB, rA, rB, TOL["fp64"], skip=True)
    assert (dA[I0] == sign * np.inf).all() and (dB[:, J0] == sign * np.inf).all()
