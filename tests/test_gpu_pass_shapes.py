"""The maxima, plane and backward passes at the sizes where their work
splits differently: rows of 16-row load groups and 64- / 256-row blocks,
columns at the width of a wave's loads, unaligned rows, plane rows taken by
one wave or one workgroup (k_pad 2048 / 2112); p* histograms whose length is
no multiple of a load; gradients whose entries use several p."""

import numpy as np
import pytest

import oracle
import test_gpu_kernels as k
from test_gpu_grad import TOL, _check, _gpu_grad
from workloads import lognormal_product

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("general_path")]

SHAPES = [
    (1, 4, 15, 3), (1, 5, 16, 4), (1, 4, 17, 255), (1, 4, 63, 257), (2, 6, 65, 256), (1, 5, 129, 513),
    (3, 4, 257, 127), (1, 7, 2048, 131), (1, 7, 2049, 62), (1, 4, 1100, 6000), (1, 4, 8190, 2047),
]


@pytest.mark.parametrize("path", ["bf16", "fp64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_scales_and_planes(gpu_lib, shape, path):
    print(f"[passes] {path} {shape}", flush=True)
    k.test_scales_and_power_planes_bit_exact(gpu_lib, ("uniform",) + shape, path, [1, 2, 4])


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(15, 3), (17, 129), (64, 255), (65, 128), (257, 127), (4100, 1030)])
def test_column_maxima_of_both_types(gpu_lib, shape, dtype):
    """c of FP64 and FP32 inputs, plain and balanced (FP64 multipliers)."""
    import torch

    kk, n = shape
    A, B = (x.astype(dtype) for x in lognormal_product(4, kk, n, seed=kk + n))
    for flags in (0, gpu_lib.FLAG_BALANCE):
        wm = gpu_lib.workspace_map(1, 4, kk, n, [1, 2], path="fp64", flags=flags)
        ws = torch.zeros(gpu_lib.workspace_size(1, 4, kk, n, [1, 2], path="fp64", flags=flags), dtype=torch.uint8,
                         device="cuda")
        gpu_lib.estimate(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), P=[1, 2], path="fp64", workspace=ws,
                         balance=bool(flags))
        c = ws.cpu().numpy()[wm["c"]:wm["c"] + 8 * n].view(np.float64)
        if flags:
            d = np.sqrt(B.astype(np.float64).max(axis=1) / A.astype(np.float64).max(axis=0))
            # a product and a quotient of the device's square root: a few FP64 roundings
            np.testing.assert_allclose(c, (B.astype(np.float64) / d[:, None]).max(axis=0), rtol=1e-15 * 4)
        else:
            np.testing.assert_array_equal(c, B.astype(np.float64).max(axis=0))


@pytest.mark.parametrize("path", ["fp64", "bf16"])
@pytest.mark.parametrize("shape", [(1, 3, 5), (5, 7, 3), (16, 32, 16), (63, 65, 64), (65, 40, 129)])
def test_gradient_with_mixed_pstar(gpu_lib, shape, path):
    """Log-normal inputs: the entries' p* differ, so some p have planes and
    some do not, also inside a 16-code load of the histogram."""
    m, kk, n = shape
    P = [1, 2, 3, 8, 64, 256]
    dt = np.float64 if path == "fp64" else np.float32
    A, B = (x.astype(dt) for x in lognormal_product(m, kk, n, seed=m * n, sigma=1.5))
    G = np.random.default_rng(m + n).standard_normal((m, n)).astype(dt)
    C, ps, dA, dB = _gpu_grad(gpu_lib, A, B, G, P, path)
    gA, gB = oracle.pnorm_grad(A, B, G, P, ps)
    _check(dA, gA, TOL[path])
    _check(dB, gB, TOL[path])
