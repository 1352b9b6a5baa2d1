"""BF16 products around the lines where the forward tile changes: 128-wide
tiles with four pipeline stages (up to 256 tiles), with two (up to 512, or a
dimension of at most 128), 256-wide tiles; fewer K steps than stages, split
p, every way through the search (top-down, a start in the family with a way
up, r = 1), tail on, off and taking everything."""

import numpy as np
import pytest

import oracle
from parity import TAU, compare_estimate
from workloads import lognormal_product

pytestmark = pytest.mark.gpu

P = [1, 2, 4, 8, 16, 32, 64, 128]

SHAPES = [
    (1, 1, 1, 1), (1, 128, 64, 128), (1, 129, 63, 127), (2, 200, 129, 150), (1, 300, 257, 400),
    (2, 1500, 192, 1450),  # 288 tiles of 128
    (260, 60, 40, 33),     # 260 tiles of one item each
    (600, 40, 65, 130),    # 1200 tiles, m <= 128
    (140, 129, 70, 129),   # 560 tiles of 128, all but one row and column padding: 256-wide
]


@pytest.fixture
def knobs(gpu_lib):
    old = gpu_lib.tail_threshold(), gpu_lib.search_start()
    yield gpu_lib
    gpu_lib.set_tail_threshold(old[0])
    gpu_lib.set_search_start(old[1])


def _check(mt, shape, tail=None, start=None, projection=None):
    import torch

    b, m, k, n = shape
    print(f"[tiles] {shape} tail={tail} start={start} {projection}", flush=True)
    if tail is not None:
        mt.set_tail_threshold(tail)
    if start is not None:
        mt.set_search_start(start)
    A, B = lognormal_product(b * m, k, n * b, seed=m + k + n)
    A = np.ascontiguousarray(A.reshape(b, m, k))
    B = np.ascontiguousarray(B.reshape(k, b, n).transpose(1, 0, 2))
    C, ps = mt.estimate(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), P=P, path="bf16", return_pstar=True,
                        projection=projection)
    ref = oracle.pnorm_estimate(A, B, P, TAU["bf16"], **({"projection": projection} if projection else {}))
    compare_estimate(C.cpu().numpy(), ps.cpu().numpy(), ref, P, "bf16",
                     **({"projection": projection} if projection else {}))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_products(knobs, shape):
    _check(knobs, shape)


@pytest.mark.parametrize("shape", [SHAPES[3], SHAPES[4], SHAPES[5]], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("way", [(0, 0, None), (65536, 0, None), (0, 3, None), (64, 6, None), (0, 0, "r1"),
                                 (300, 0, "r1")], ids=str)
def test_ways_through_the_search(knobs, shape, way):
    _check(knobs, shape, *way)
