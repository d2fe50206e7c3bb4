"""The iteration's statistics where their kernels branch: one block up to 16,384 angles, histograms
and gathered candidates above; epilogue blocks of 64 queries up to 32,768 points, 256 above. The
references are NumPy's sort and means of the angles between the normals before and after."""
import numpy as np
import pytest
import torch

from paper_2405_13839_amd import synth
from tests.helpers import cuda, host, unit_rows

pytestmark = pytest.mark.gpu


def _angles(a, b):
    ch = np.linalg.norm(b.astype(np.float64) - a.astype(np.float64), axis=0)
    return np.degrees(2 * np.arcsin(np.minimum(1, ch / 2))), ch


@pytest.mark.parametrize("n", [2, 63, 1025, 16_384, 16_385, 32_768, 32_769, 200_003])
@pytest.mark.parametrize("frac", [1e-9, 0.01, 0.37, 1.0])
def test_top_mean_is_the_sorted_mean(n, frac):
    from paper_2405_13839_amd import dwg
    c = synth.torus_ellipsoids(max(n, 64), seed=9)
    P, area = cuda(c.P[:, :n]), cuda(c.area[:n])
    N = cuda(unit_rows(np.random.default_rng(n), n))
    prm = dwg.Params(lam=10.0, beta=2.3)
    w = host(dwg.gwn(P, N, area, None, P, prm)[0]).astype(np.float64)
    before = host(N)
    _, st = dwg.iterate(P, area, None, N, prm, max_iters=1, fixed_iters=True, top_frac=frac)
    th, ch = _angles(before, host(N))
    k = dwg.top_count(n, frac)
    np.testing.assert_allclose(st[0, 1].item(), np.sort(th)[::-1][:k].mean(), rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(st[0, 2].item(), ch.mean(), rtol=1e-12)
    np.testing.assert_allclose(st[0, 0].item(), w.mean(), rtol=1e-9, atol=1e-12 * np.abs(w).max())


@pytest.mark.parametrize("n", [100, 16_384, 16_385, 70_000])
def test_all_angles_equal(n):
    """Zero weights leave every normal, so that all angles tie at 0 (more ties than candidates are
    gathered, for the larger counts)."""
    from paper_2405_13839_amd import dwg
    P = cuda(np.random.default_rng(1).standard_normal((3, n)))
    N = cuda(unit_rows(np.random.default_rng(2), n))
    before = N.clone()
    _, st = dwg.iterate(P, torch.zeros(n, device="cuda"), None, N, dwg.Params(beta=2.3), max_iters=1, fixed_iters=True)
    assert st[0, 0].item() == 0.0 and st[0, 1].item() == 0.0 and torch.equal(N, before)


def test_few_points_move_among_many_that_do_not():
    """Nearly all angles 0, the k-th largest among them or among the few others."""
    from paper_2405_13839_amd import dwg
    n = 50_000
    rng = np.random.default_rng(5)
    P = rng.uniform(-1, 1, (3, n)).astype(np.float32)
    P[:, :] = P[:, :1]  # coincident pairs contribute nothing
    P[:, :300] += rng.uniform(0.5, 1.5, (3, 300)).astype(np.float32)
    area = np.zeros(n, np.float32)
    area[:300] = 1.0
    N = cuda(unit_rows(rng, n))
    for frac in (0.001, 0.004, 0.02, 0.5):
        before = host(N)
        _, st = dwg.iterate(cuda(P), cuda(area), None, N, dwg.Params(), max_iters=1, fixed_iters=True, top_frac=frac)
        th, _ = _angles(before, host(N))
        want = np.sort(th)[::-1][:dwg.top_count(n, frac)].mean()
        np.testing.assert_allclose(st[0, 1].item(), want, rtol=1e-12, atol=1e-12)
