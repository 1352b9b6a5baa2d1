"""The 256-wide BF16 tiles at few K steps (plain steps of 64, split ones of
32 inner indices): their loop keeps the loads of two steps on the way, so the
first, second and last steps differ from the rest.  Against the oracle at the
BF16 path's tolerance; the tail off, so that every p runs densely."""

import numpy as np
import pytest

import oracle
from parity import TAU, compare_estimate
from workloads import lognormal_product

pytestmark = pytest.mark.gpu

P = [1, 2, 4, 8, 16, 32, 64, 128]


@pytest.mark.parametrize("k", [1, 64, 65, 130, 190, 250, 321])
@pytest.mark.parametrize("projection", [None, "r1"])
def test_few_k_steps(gpu_lib, k, projection):
    import torch

    m, n = 2820, 3080  # 23 x 25 tiles of 128: more than the 128-wide kernels take
    A, B = lognormal_product(m, k, n, seed=k)
    old = gpu_lib.tail_threshold()
    gpu_lib.set_tail_threshold(0)
    try:
        C, ps = gpu_lib.estimate(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), P=P, path="bf16",
                                 projection=projection, return_pstar=True)
    finally:
        gpu_lib.set_tail_threshold(old)
    ref = oracle.pnorm_estimate(A.astype(np.float64), B.astype(np.float64), P, TAU["bf16"], projection=projection)
    compare_estimate(C.cpu().numpy(), ps.cpu().numpy(), ref, P, "bf16", projection=projection)
