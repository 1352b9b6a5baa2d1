"""The work and the device time of APSP's squarings under the GEMM's name,
whichever launch runs them: undirected and directed graphs, in 128-wide tiles,
the launch of them beside 256-wide ones, and 256-wide tiles."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2100, 3100, 4200])
@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("projection", [None, "r1"])
def test_squarings_are_counted(gpu_lib, n, directed, projection):
    import torch

    rng = np.random.default_rng(n)
    W = rng.uniform(0.0, 3.0, (n, n)).astype(np.float32)
    if not directed:
        W = np.minimum(W, W.T)
    print(f"[apsp timing] {n} directed={directed} {projection}", flush=True)
    Wd = torch.from_numpy(W).cuda()
    gpu_lib.timing_reset()
    gpu_lib.timing_enable(True)
    try:
        gpu_lib.apsp(Wd, P=[1, 2, 4, 8, 16], path="bf16", n_squarings=3, projection=projection)
        work = gpu_lib.timing_work("mt_pfamily_gemm_bf16")
        ms, launches = gpu_lib.timing_span("mt_pfamily_gemm_bf16")
    finally:
        gpu_lib.timing_enable(False)
        gpu_lib.timing_reset()
    # three squarings of at least one p over the triangle (the whole matrix where directed)
    assert launches == 3 and ms > 0.0
    assert work >= 3 * 2.0 * n ** 3 / (1 if directed else 2)
