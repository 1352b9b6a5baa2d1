"""On the BF16 path the r = 1 projection takes the plain estimate's workspace
size, also where the two run on tiles of different sides: a workspace sized
for one serves the other (no GPU needed)."""

import os

import pytest

import paper_1511_05690_amd as mt

pytestmark = pytest.mark.skipif(not os.path.exists(mt.library_path()), reason="libmaxtimes.so not built")

P = [1, 2, 4, 8, 16, 32, 64, 128]


@pytest.mark.parametrize("shape", [(1, 64, 64, 64), (1, 1500, 2050, 1777), (1, 2100, 700, 2100), (1, 40, 300, 110000),
                                   (300, 129, 70, 129), (16, 600, 80, 500), (1, 5000, 64, 5000)],
                         ids=lambda s: "x".join(map(str, s)))
def test_product(shape):
    assert mt.workspace_size(*shape, P, flags=mt.FLAG_PROJECT_R1) == mt.workspace_size(*shape, P)


@pytest.mark.parametrize("n", [1, 700, 2048, 2049, 2500, 2880, 2900, 3500, 5000])
def test_apsp(n):
    assert mt.apsp_workspace_size(n, P, path="bf16", flags=mt.FLAG_PROJECT_R1) == mt.apsp_workspace_size(n, P, path="bf16")
