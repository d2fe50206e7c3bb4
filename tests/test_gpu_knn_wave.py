"""The wavefront pass of the neighbour search where its parts meet: rows of cells with more and fewer
points than a wavefront, batches that are merged and candidates inserted one by one, lists from 1
to 16 long, references in one place. Coordinates are small whole numbers, so squared distances are
exact and equal ones are common: the answer is the k smallest (distance, index) pairs, exactly."""
import numpy as np
import pytest

from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu


def _expect(R, Q, k):
    d2 = ((R[:, None, :] - Q[:, :, None]) ** 2).sum(axis=0)
    idx = np.argsort(d2, axis=1, kind="stable")[:, :k]
    return idx, np.sqrt(np.take_along_axis(d2, idx, axis=1))


@pytest.mark.parametrize("n", [17, 63, 64, 65, 500, 5000])
@pytest.mark.parametrize("k", [1, 2, 12, 13, 15, 16])
@pytest.mark.parametrize("kind", ["box", "plane", "place"])
def test_far_queries_find_the_nearest(n, k, kind):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n * 17 + k)
    R = rng.integers(0, 24, (3, n)).astype(np.float64)
    if kind == "plane":
        R[2] = 3
    if kind == "place":
        R[:, n // 4:] = R[:, :1]
    Q = rng.integers(-60, 90, (3, 400)).astype(np.float64)
    Q[:, :100] = R[:, rng.integers(0, n, 100)] + rng.integers(-9, 10, (3, 100))
    idx, dist = dwg.knn(cuda(R.astype(np.float32)), cuda(Q.astype(np.float32)), k)
    want, wdist = _expect(R, Q, k)
    np.testing.assert_array_equal(host(idx).astype(np.int64).reshape(want.shape), want)
    np.testing.assert_allclose(host(dist).reshape(want.shape), wdist, rtol=2e-7)
