"""The BF16 forward's 128-wide tiles end where a launch could not hold one
workgroup of 512 threads for each (2^32 threads); 256-wide tiles go on to
twice the columns (no GPU needed: the padded sizes show the tile)."""

import os

import pytest

import paper_1511_05690_amd as mt

pytestmark = pytest.mark.skipif(not os.path.exists(mt.library_path()), reason="libmaxtimes.so not built")


@pytest.mark.parametrize("m,n", [(1, 1 << 24), (1 << 24, 100)])
def test_largest_launch(m, n):
    for b, side in ((63, 128), (64, 256), (127, 256)):
        w = mt.workspace_map(b, m, 1, n, [1, 2], flags=mt.FLAG_PROJECT_R1)
        assert w["m_pad"] * w["n_pad"] == side * (1 << 24)
        assert b * (w["m_pad"] // side) * (w["n_pad"] // side) * 512 < 1 << 32
