"""Exact neighbour lists where the grid search branches: reference counts around the one-block
build (8,192) and the sample (4,096), query counts around the cell-order sort (16,384), own and
foreign queries, the smallest and largest k. Coordinates are multiples of 1/64, so squared
distances are exact in float32 and most are tied: the lists must equal brute force's by
(squared distance, index) element by element."""
import numpy as np
import pytest
import torch

from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu


def _brute(R, Q, k, own):
    """Indices and distances by float64 arithmetic, ordered by (squared distance, index); own: the
    reference that each query is, left out."""
    idx, dist = [], []
    for s in range(0, Q.shape[1], 512):
        d2 = ((Q[:, s:s + 512, None].astype(np.float64) - R[:, None, :]) ** 2).sum(0)
        if own is not None:
            d2[np.arange(d2.shape[0]), own[s:s + 512]] = np.inf
        o = np.argsort(d2, axis=1, kind="stable")[:, :k]
        idx.append(o)
        dist.append(np.sqrt(np.take_along_axis(d2, o, 1)))
    return np.concatenate(idx), np.concatenate(dist)


def _cloud(kind, n, rng):
    if kind == "raster":  # a scan stored row by row, 256 points to a row
        i = np.arange(n)
        p = np.stack([i % 256, i // 256, (i % 256) // 16]).astype(np.float64)
    elif kind == "ball":
        p = rng.integers(-30, 31, (3, n)).astype(np.float64)
    else:  # "clumps": two tight clumps with repeated points and a few points far away
        p = rng.integers(-3, 4, (3, n)).astype(np.float64) + np.where(np.arange(n) % 2, 400.0, 0.0)
        p[:, ::997] *= 50.0
    return np.ascontiguousarray((p / 64.0).astype(np.float32))


@pytest.mark.parametrize("kind", ["raster", "ball", "clumps"])
@pytest.mark.parametrize("nr,k", [(17, 16), (4095, 1), (4097, 10), (8192, 16), (8193, 7), (20_001, 16)])
def test_own_neighbours_exact(kind, nr, k):
    from paper_2405_13839_amd import dwg
    R = _cloud(kind, nr, np.random.default_rng(nr + k))
    Rc = cuda(R)
    idx, dist = dwg.knn(Rc, Rc, k, self_skip=True)
    sel = np.unique(np.concatenate([np.arange(min(nr, 200)), np.arange(0, nr, 41), [nr - 1]]))
    bi, bd = _brute(R, R[:, sel], k, sel)
    np.testing.assert_array_equal(host(idx)[sel], bi)
    np.testing.assert_array_equal(host(dist)[sel], bd.astype(np.float32))
    # the kernel radius that the search writes without the lists: the mean of the same distances
    mean = host(dist).astype(np.float64).mean(1)
    np.testing.assert_allclose(host(dwg.delta_knn_mean(Rc, k)), mean, rtol=k * 2.0 ** -23, atol=0)


@pytest.mark.parametrize("nr,m,k", [(16, 1, 16), (300, 16_383, 10), (300, 16_384, 10), (9000, 24_577, 16)])
def test_foreign_neighbours_exact(nr, m, k):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(nr + m)
    R = _cloud("ball", nr, rng)
    Q = _cloud("ball", m, rng)
    Q[:, ::53] *= 8.0  # outside the grid, searched by a wavefront each
    idx, dist = dwg.knn(cuda(R), cuda(Q), k)
    sel = np.arange(0, m, max(1, m // 700))
    bi, bd = _brute(R, Q[:, sel], k, None)
    np.testing.assert_array_equal(host(idx)[sel], bi)
    np.testing.assert_array_equal(host(dist)[sel], bd.astype(np.float32))
    assert torch.isfinite(dist).all()
