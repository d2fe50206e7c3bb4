"""NaN points in a cloud: the neighbour lists of such points have no entries, and nothing is read by
them. The results of the other points are those of the cloud without the NaN points, bit for bit (fewer
than 8,192 points: every point is an anchor of the features)."""
import numpy as np
import pytest
import torch

from paper_2405_13839_amd import mlp_init
from tests.helpers import cuda, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bad", [(3000, 1), (3000, 700), (40, 20)])
def test_other_points_do_not_see_them(n, bad):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n + bad)
    P = unit_rows(rng, n) + rng.uniform(-0.01, 0.01, (3, n)).astype(np.float32)
    where = rng.choice(n, bad, replace=False)
    P[rng.integers(0, 3, bad), where] = np.nan
    good = torch.from_numpy(np.setdiff1d(np.arange(n), where)).cuda()
    A, B = cuda(P), cuda(P)[:, good].contiguous()
    prm = cuda(mlp_init.init_params(3))
    assert torch.equal(dwg.pca_normals(A)[:, good], dwg.pca_normals(B))
    assert torch.equal(dwg.voronoi_area(A)[good], dwg.voronoi_area(B))
    assert torch.equal(dwg.features(A)[good], dwg.features(B))
    assert torch.equal(dwg.mlp_normals(A, prm)[:, good], dwg.mlp_normals(B, prm))
    assert torch.equal(dwg.delta_knn_mean(A)[good], dwg.delta_knn_mean(B))


def test_too_few_points_that_are_not_nan():
    """Five neighbours where sixteen are asked for: the lists' other entries are left out."""
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(7)
    P = np.full((3, 200), np.nan, np.float32)
    P[:, 10:16] = rng.uniform(-1, 1, (3, 6))
    A = cuda(P)
    idx, dist = dwg.knn(A, A, 16, self_skip=True)
    assert bool(torch.isfinite(dist[10:16, :5]).all()) and bool(torch.isinf(dist[10:16, 5:]).all())
    nv = dwg.pca_normals(A)[:, 10:16]
    assert bool(torch.isfinite(nv).all()) and torch.allclose(nv.norm(dim=0), torch.ones(6, device="cuda"))
    assert bool((dwg.voronoi_area(A)[10:16] > 0).all())
    assert dwg.features(A).shape == (200, 48) and dwg.mlp_normals(A, cuda(mlp_init.init_params(3))).shape == (3, 200)
    torch.cuda.synchronize()
