"""References that are NaN, whatever their bits, are nobody's neighbours: not in the thread-per-query pass
and not in the wavefront pass (queries far from the cloud)."""
import numpy as np
import pytest

from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [0x7FC00000, 0x7F800001, 0xFFC00000, 0xFFF00000, 0xFFFFFFFF])
@pytest.mark.parametrize("nr,k", [(600, 1), (600, 16), (9000, 10)])
def test_nan_references_are_never_taken(nr, k, bits):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(nr + k)
    R = (rng.integers(-60, 61, (3, nr)) / 64.0).astype(np.float32)
    bad = rng.choice(nr, nr // 20, replace=False)
    R.view(np.uint32)[:, bad] = bits
    good = np.setdiff1d(np.arange(nr), bad)
    Q = (rng.integers(-60, 61, (3, 400)) / 64.0).astype(np.float32)
    Q[:, ::5] *= 8.0
    d2 = ((Q[:, :, None].astype(np.float64) - R[:, None, good]) ** 2).sum(0)
    o = np.argsort(d2, axis=1, kind="stable")[:, :k]
    idx, dist = dwg.knn(cuda(R), cuda(Q), k)
    np.testing.assert_array_equal(host(idx), good[o])
    np.testing.assert_array_equal(host(dist), np.sqrt(np.take_along_axis(d2, o, 1)).astype(np.float32))
