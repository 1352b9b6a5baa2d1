"""APSP of undirected graphs on the BF16 path (upper triangle and mirrored
outputs) where the distances span the family: entries decided at every p, the
split ones (1, 2, 4) among them, and none, in 128-wide tiles (n = 2100), the
launch of them beside 256-wide ones (n = 3100) and 256-wide tiles (n = 4200),
along every way through the search and with the tail off, at small and set
thresholds and taking everything.  X and p* stay their own transposes to the
last bit, also inside the diagonal's tiles, and agree with the oracle's
squaring of the X before on rows at the edges of tiles (bars of parity.py)."""

import numpy as np
import pytest

import oracle
from parity import TAU, compare_estimate

pytestmark = pytest.mark.gpu

P = [1, 2, 4, 8, 16, 32, 64, 128]
_X0, _REF = {}, {}


@pytest.fixture
def knobs(gpu_lib):
    old = gpu_lib.tail_threshold(), gpu_lib.search_start()
    yield gpu_lib
    gpu_lib.set_tail_threshold(old[0])
    gpu_lib.set_search_start(old[1])


def _graph(n):
    """About 24 neighbours per vertex, weights 40 u^2: one and two hops span
    distances from 0 to 80, unstable at p = 1 beyond 69."""
    rng = np.random.default_rng(n)
    edge = rng.random((n, n)) < 24.0 / n
    W = np.where(edge, 40.0 * rng.random((n, n)) ** 2, np.inf).astype(np.float32)
    W = np.triu(W, 1)
    W = np.where(np.tri(n, dtype=bool), np.float32(np.inf), W)
    W = np.minimum(W, W.T)
    np.fill_diagonal(W, 0.0)
    return W


def _rows(n):
    return np.array([r for r in (0, 1, 63, 64, 127, 128, 129, 255, 256, 257, 511, 512, 1000, 1279, 1280, 2047, 2048,
                                 2431, 2432, 3071, 3072, 4095, 4096, n - 2, n - 1) if r < n])


def _oracle(X, rows, projection):
    return oracle.pnorm_estimate_rows(X, X, P, TAU["bf16"], rows, projection=projection)


def _squarings(mt, n, T, projection=None):
    import torch

    X, ps = mt.apsp(torch.from_numpy(_graph(n)).cuda(), s=1.0, P=P, path="bf16", n_squarings=T, raw=True,
                    projection=projection, return_pstar=True)
    assert torch.equal(X, X.T) and (T == 0 or torch.equal(ps, ps.T))
    return X.cpu().numpy(), ps.cpu().numpy()


def _compare(X, ps, ref, n, projection):
    rows = _rows(n)
    skip = np.zeros((len(rows), n), dtype=bool)
    skip[np.arange(len(rows)), rows] = True
    print(compare_estimate(X[rows], ps[rows], ref, P, "bf16", projection=projection, clamp=True, skip=skip), flush=True)


# (search start, tail threshold, projection); -1: the pilot's start, None: the default threshold
WAYS = [(-1, None, None), (0, 0, None), (0, 65536, None), (0, 3, None), (3, None, None), (5, 300, None), (6, 65536, None),
        (7, 0, None), (-1, None, "r1"), (-1, 0, "r1"), (-1, 65536, "r1"), (-1, 2, "r1")]


@pytest.mark.parametrize("n", [2100, 3100, 4200])
@pytest.mark.parametrize("start,tail,projection", WAYS)
def test_first_squaring(knobs, n, start, tail, projection):
    print(f"[apsp sym] n={n} start={start} tail={tail} {projection}", flush=True)
    if n not in _X0:
        _X0[n] = _squarings(knobs, n, 0)[0]
    if (n, projection) not in _REF:
        _REF[n, projection] = _oracle(_X0[n], _rows(n), projection)
    ref = _REF[n, projection]
    assert set(range(len(P))) | {255} <= set(np.unique(ref["pstar_idx"]))
    knobs.set_search_start(start)
    if tail is not None:
        knobs.set_tail_threshold(tail)
    X, ps = _squarings(knobs, n, 1, projection)
    _compare(X, ps, ref, n, projection)


@pytest.mark.parametrize("n,projection", [(2100, None), (3100, "r1"), (4200, None)])
def test_second_squaring(gpu_lib, n, projection):
    print(f"[apsp sym] second squaring n={n} {projection}", flush=True)
    X1, _ = _squarings(gpu_lib, n, 1, projection)
    X2, ps = _squarings(gpu_lib, n, 2, projection)
    ref = _oracle(X1, _rows(n), projection)
    assert set(range(1, len(P))) <= set(np.unique(ref["pstar_idx"]))
    _compare(X2, ps, ref, n, projection)
