"""FP64 APSP squarings whose entries leave the dense search: deferred planes
reached off the pilot's sample, entries with no path (S exactly 0), entries
whose S underflows at the larger p and is stable at a smaller one, rows of one
to several tail entries.  Against the same squarings with the tail and the
deferred planes off; the recorded S differ by the order of FP64 sums only
(n terms: at most n 2^-53 relative, under the 1/p root), p* not at all."""

import numpy as np
import pytest

from workloads import er_graph

pytestmark = pytest.mark.gpu

P = [1, 2, 4, 8, 16, 32, 64, 128, 256, 512]


@pytest.fixture
def knobs(gpu_lib):
    old = gpu_lib.tail_threshold(), gpu_lib.deferred_planes()
    yield gpu_lib
    gpu_lib.set_tail_threshold(old[0])
    gpu_lib.set_deferred_planes(old[1])


def _both(mt, W, T, tail):
    import torch

    Wd = torch.from_numpy(W).cuda()

    def go(tail, deferred):
        mt.set_tail_threshold(tail)
        mt.set_deferred_planes(deferred)
        X, ps = mt.apsp(Wd, s=1.0, P=P, path="fp64", n_squarings=T, raw=True, return_pstar=True,
                        out_dtype=torch.float64)
        return X.cpu().numpy(), ps.cpu().numpy()

    X, ps = go(tail, True)
    X0, ps0 = go(0, False)
    np.testing.assert_array_equal(ps, ps0)
    np.testing.assert_allclose(X, X0, rtol=4 * W.shape[0] * 2.0 ** -53, atol=0)
    return X, ps


def _near_complete(n, seed):
    rng = np.random.default_rng(seed)
    W = rng.uniform(0.05, 0.5, (n, n)).astype(np.float32)
    np.fill_diagonal(W, 0.0)
    return W


@pytest.mark.parametrize("far", [1, 7, 70])
@pytest.mark.parametrize("tail", [512, 64])
def test_deferred_planes_off_the_sample(knobs, far, tail):
    """Vertices at distance 60 (p* = 8, below the three largest p), none of
    them in the pilot's 64 sampled rows or columns."""
    n = 2080
    sampled = {((2 * q + 1) * n) // 128 for q in range(64)}
    W = _near_complete(n, far)
    lone = [v for v in range(100, n, 2) if v not in sampled][:far]
    for v in lone:
        W[v, :] = np.float32(60.0)
        W[:, v] = np.float32(60.0)
        W[v, v] = 0.0
    print(f"[apsp tail] far={far} tail={tail}", flush=True)
    X, ps = _both(knobs, W, 2, tail)
    off = [v for v in range(n) if v not in lone]
    assert (ps[np.ix_(lone, off)] == P.index(8)).all()


@pytest.mark.parametrize("prob,T", [(0.003, 1), (0.003, 3), (0.0004, 2)])
def test_sparse_graphs(knobs, prob, T):
    """Unreachable pairs (zeros in X) and long distances."""
    W = er_graph(2049, prob, 10.0, seed=int(prob * 1e5) + T)
    print(f"[apsp tail] prob={prob} T={T}", flush=True)
    X, ps = _both(knobs, W, T, 4096)
    assert (X == 0).any() and len(np.unique(ps)) > 4


@pytest.mark.parametrize("weight", [1.4, 1.6, 3.1, 13.0, 200.0])
def test_underflow_at_the_larger_p(knobs, weight):
    """A few entries per row at a distance where S at the larger p is exactly
    0 or below tau, the rest close by."""
    n = 2048
    W = _near_complete(n, 3)
    rng = np.random.default_rng(int(weight * 10))
    cut = rng.choice(n, 5, replace=False)
    W[:, cut] = np.float32(weight)
    np.fill_diagonal(W, 0.0)
    print(f"[apsp tail] weight={weight}", flush=True)
    _both(knobs, W, 1, 512)
