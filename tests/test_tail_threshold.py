"""The sparse tail's threshold as state: what the getter returns can be set
back without a change of any workspace size, and the limit of 128-wide tiles
(128 entries at the default of 512) is that of the tiles that run."""

import os

import numpy as np
import pytest

import oracle
import paper_1511_05690_amd as mt
from parity import TAU, compare_estimate

P = [1, 2, 4, 8, 16, 32, 64, 128]

built = pytest.mark.skipif(not os.path.exists(mt.library_path()), reason="libmaxtimes.so not built")


@built
def test_set_what_was_read():
    def sizes():
        return [mt.workspace_size(b, m, k, n, P, path=path)
                for path in ("bf16", "fp64")
                for b, m, k, n in ((1, 257, 513, 255), (1, 1500, 2050, 1777), (16, 100, 600, 90), (1, 4096, 512, 4096))
                ] + [mt.apsp_workspace_size(n, P, path=path) for path in ("bf16", "fp64") for n in (700, 3500)]

    old = mt.tail_threshold()
    before = sizes()
    mt.set_tail_threshold(mt.tail_threshold())
    assert sizes() == before and mt.tail_threshold() == old
    try:
        for thr in (0, 3, 300, 65536):
            mt.set_tail_threshold(thr)
            assert mt.tail_threshold() == thr
    finally:
        mt.set_tail_threshold(old)
    assert sizes() == before


@pytest.mark.gpu
@pytest.mark.parametrize("threshold,left,handed", [(None, 100, True), (None, 200, False), (256, 200, True),
                                                   (3, 5, False), (5, 5, True)])
def test_limit_of_a_128_wide_tile(gpu_lib, threshold, left, handed):
    """512^3 is 16 tiles of 128.  `left` entries of the first have one term of
    1e-20 in a row of 1e-40 and need p = 1, all others are stable at the
    largest p: the tile stops there when it hands them over."""
    import torch

    rng = np.random.default_rng(21)
    n = 512
    A = rng.uniform(0.9, 1.0, (n, n)).astype(np.float32)
    B = rng.uniform(0.9, 1.0, (n, n)).astype(np.float32)
    high = A.copy(), B.copy()
    for i in range(5):
        A[i], A[i, i], B[i] = 1e-20, 1.0, 1.0
        B[i, :left // 5] = 1e-20

    def run(A, B):
        gpu_lib.timing_reset()
        gpu_lib.timing_enable(True)
        try:
            C, ps = gpu_lib.estimate(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), P=P, path="bf16",
                                     return_pstar=True)
            return C.cpu().numpy(), ps.cpu().numpy(), gpu_lib.timing_work("mt_pfamily_gemm_bf16")
        finally:
            gpu_lib.timing_enable(False)
            gpu_lib.timing_reset()

    print(f"[tail] threshold {threshold}, {left} left", flush=True)
    old = gpu_lib.tail_threshold()
    if threshold is not None:
        gpu_lib.set_tail_threshold(threshold)
    try:
        work_high = run(*high)[2]
        C, ps, work = run(A, B)
    finally:
        gpu_lib.set_tail_threshold(old)
    ref = oracle.pnorm_estimate(A, B, P, TAU["bf16"])
    assert (ref["pstar_idx"] != len(P) - 1).sum() == left
    compare_estimate(C, ps, ref, P, "bf16")
    assert (work == work_high) == handed
