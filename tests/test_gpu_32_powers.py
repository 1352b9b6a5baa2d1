"""Families of 32 powers, the most the ABI accepts, through every route that
writes power planes: products on both paths (row maxima taken with the planes
by a wave or by a workgroup, and apart), deferred planes, planes all split,
the backward with the last power in use, the r = 2 projection whose family and
added norms are 32 together, and APSP.  Bars: tests/parity.py and
test_gpu_grad.py."""

import math

import numpy as np
import pytest

import oracle
from parity import TAU, compare_estimate
from test_gpu_grad import TOL, _check, _gpu_grad
from workloads import er_graph, gradient_case, lognormal_product, rgg_graph

pytestmark = pytest.mark.gpu

P32 = list(range(1, 21)) + [24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024]
# eight powers of two (the r = 2 projection adds 3, 6, 12, 24, 48 and 96) and
# eighteen odd ones: 32 with the added norms
P26 = sorted([1, 2, 4, 8, 16, 32, 64, 128] + list(range(5, 40, 2)))


def _dev(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("shape", [(5, 70, 9), (200, 300, 100), (130, 2100, 70)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("path", ["bf16", "fp64"])
def test_products(general_path, path, dtype, shape):
    m, k, n = shape
    print(f"[32 powers] {path} {dtype.__name__} {shape}", flush=True)
    A, B = lognormal_product(m, k, n, seed=m + k, dtype=dtype)
    C, ps = general_path.estimate(_dev(A), _dev(B), P=P32, path=path, return_pstar=True)
    ref = oracle.pnorm_estimate(A, B, P32, TAU[path])
    compare_estimate(C.cpu().numpy(), ps.cpu().numpy(), ref, P32, path)


@pytest.mark.parametrize("path", ["bf16", "fp64"])
def test_deferred_planes(gpu_lib, path):
    """2^22 outputs: the pilot steers the search and the planes of the smaller
    p are written late (the mask of the early ones ends at power 31)."""
    n, k = 2048, 300
    print(f"[32 powers] deferred {path}", flush=True)
    dt = np.float64 if path == "fp64" else np.float32
    A, B = lognormal_product(n, k, n, seed=32, dtype=dt)
    A[700:704, 1:] = dt(0)  # p* of these rows follows B's first row alone
    C, ps = gpu_lib.estimate(_dev(A), _dev(B), P=P32, path=path, return_pstar=True)
    rows = np.r_[0:20, 690:710, 2030:2048]
    ref = oracle.pnorm_estimate_rows(A, B, P32, TAU[path], rows)
    compare_estimate(C.cpu().numpy()[rows], ps.cpu().numpy()[rows], ref, P32, path)


@pytest.mark.parametrize("path", ["bf16", "fp64"])
@pytest.mark.parametrize("P", [list(range(1, 33)), list(range(1, 64, 2))], ids=["1..32", "odd"])
def test_backward(general_path, path, P):
    """Every power split on the BF16 path; p* spread over the family, its last
    power in use."""
    dt = np.float64 if path == "fp64" else np.float32
    G = gradient_case(1, 70, 90, 130, seed=7, dtype=dt)[2][0]
    A, B = lognormal_product(70, 90, 130, seed=7, sigma=12.0 if path == "fp64" else 2.0,
                             clip=1e40 if path == "fp64" else 1e6, dtype=dt)
    print(f"[32 powers] backward {path}", flush=True)
    _, ps, dA, dB = _gpu_grad(general_path, A, B, G, P, path)
    assert (ps == 31).any() and len(np.unique(ps)) > 4
    rA, rB = oracle.pnorm_grad(A, B, G, P, ps)
    _check(dA, rA, TOL[path])
    _check(dB, rB, TOL[path])


def test_r2_with_added_norms(gpu_lib):
    A, B = lognormal_product(60, 90, 50, seed=3, dtype=np.float64)
    assert len(P26) + len(oracle.pnorm.r2_aux_powers(P26)) == 32
    print("[32 powers] r2", flush=True)
    C, ps = gpu_lib.estimate(_dev(A), _dev(B), P=P26, path="fp64", return_pstar=True, projection="r2")
    ref = oracle.pnorm_estimate(A, B, P26, TAU["fp64"], projection="r2")
    compare_estimate(C.cpu().numpy(), ps.cpu().numpy(), ref, P26, "fp64", projection="r2")


@pytest.mark.parametrize("path", ["bf16", "fp64"])
def test_apsp(gpu_lib, path):
    import torch

    n = 200
    print(f"[32 powers] apsp {path}", flush=True)
    if path == "fp64":
        W, s, T = er_graph(n, 0.04, 10.0, seed=901), 1.0, 3
    else:
        W, s, T = rgg_graph(n, math.sqrt(20.0 / (math.pi * n)), 100.0, seed=902), 0.35, 1
    ref = oracle.apsp_estimate(W, s, P32, TAU[path], T=T)["X"]
    X = gpu_lib.apsp(_dev(W), s=s, P=P32, path=path, n_squarings=T, raw=True, out_dtype=torch.float64).cpu().numpy()
    assert ((X == 0) == (ref == 0)).all()
    assert (np.abs(X - ref) / np.maximum(ref, 1e-300)).max() <= {"fp64": 1e-5, "bf16": 2e-3}[path]
