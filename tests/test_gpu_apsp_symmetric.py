"""APSP of undirected graphs on the BF16 path: only the tiles on and above the
diagonal run and their outputs are mirrored, with 128-wide tiles (n = 2100),
in a launch beside the 256-wide one (n = 3100) and with 256-wide tiles (n =
4200).  X and p* are their own transposes, and agree with the general path,
which the same graph takes once one edge's two directions differ by one part
in 2^20 (at most 1.1e-5 in X, weights up to 30).  Tolerance: the two sum the
same positive terms in FP32 (at the split p in another order), n 2^-24
relative on a ring result each, twice that on the ratio of the r = 1
projection, for every squaring and once for the changed edge; entries with different p* (a ring result within that of tau) at
most one in 10^4."""

import numpy as np
import pytest

from workloads import dense_graph, rgg_graph

pytestmark = pytest.mark.gpu

P = [1, 2, 4, 8, 16, 32, 64, 128]


def _graph(kind, n):
    if kind == "rgg":
        return rgg_graph(n, 1.6 / np.sqrt(n), 100.0, seed=n)
    W = dense_graph(n, 0.5, 30.0, seed=n)
    return np.minimum(W, W.T)


@pytest.mark.parametrize("n", [2100, 3100, 4200])
@pytest.mark.parametrize("kind,projection", [("rgg", "r1"), ("rgg", None), ("dense", "r1"), ("dense", None)])
def test_upper_triangle(gpu_lib, n, kind, projection):
    import torch

    T = 2
    W = _graph(kind, n)
    assert (W == W.T).all()
    V = W.copy()
    i, j = np.argwhere(np.isfinite(W) & (W > 0))[n // 2]
    V[i, j] *= np.float32(1 + 2.0 ** -20)
    out = []
    for G in (W, V):
        X0 = gpu_lib.apsp(torch.from_numpy(G).cuda(), s=0.35, P=P, path="bf16", n_squarings=0, raw=True)
        assert torch.equal(X0, X0.T) == (G is W)
        X, ps = gpu_lib.apsp(torch.from_numpy(G).cuda(), s=0.35, P=P, path="bf16", n_squarings=T, raw=True,
                             projection=projection, return_pstar=True)
        out.append((X, ps))
    (X, ps), (Y, qs) = out
    assert torch.equal(X, X.T) and torch.equal(ps, ps.T)
    same = ps == qs
    assert int((~same).sum()) <= n * n // 10 ** 4
    tol = (2 * T + 2) * n * 2.0 ** -24
    rel = ((X - Y).abs() / Y.clamp_min(1e-37))[same & (Y > 0)]
    print(f"   {kind} {n} {projection}: max rel {float(rel.max()):.1e} of {tol:.1e}, "
          f"p* differ at {int((~same).sum())}", flush=True)
    assert float(rel.max()) <= tol
    assert torch.equal((X == 0)[same], (Y == 0)[same])
