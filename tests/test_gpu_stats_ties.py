"""The convergence statistic where more angles share their leading 28 bits than one block holds (16,384):
up to 32,768 angles by one block, above by histograms of the other 36 bits. Most points have no
weight, so that their start normals can be chosen freely: at one angle from the field's normal, but for the
rounding of their components (a spread of about 1e-7, all in one bucket), or at two. The
reference is NumPy's sort of the angles between the normals before and after."""
import numpy as np
import pytest
import torch

from tests.helpers import cuda, host, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32_768, 32_769, 70_001, 300_007])
@pytest.mark.parametrize("angles", [(0.3,), (1e-3,), (0.5, 0.5000001), (0.0,)])
def test_many_angles_in_one_bucket(n, angles):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n)
    P = rng.uniform(-1, 1, (3, n)).astype(np.float32)
    P[:, 300:] += 4.0
    area = np.zeros(n, np.float32)
    area[:300] = 1.0
    N = unit_rows(rng, n)
    prm = dwg.Params(beta=2.3)
    Pc, ac = cuda(P), cuda(area)
    g = host(dwg.gwn(Pc, cuda(N), ac, None, Pc, prm)[1]).astype(np.float64)
    new = -g / np.linalg.norm(g, axis=0)
    t = np.cross(new.T, rng.standard_normal((n, 3))).T
    t /= np.linalg.norm(t, axis=0)
    at = np.asarray(angles)[rng.integers(0, len(angles), n)]
    N[:, 300:] = (np.cos(at) * new + np.sin(at) * t)[:, 300:]
    before = cuda(N)
    for frac in (1e-9, 0.003, 0.01, 0.37, 0.6, 1.0):
        M = before.clone()
        _, st = dwg.iterate(Pc, ac, None, M, prm, max_iters=1, fixed_iters=True, top_frac=frac)
        ch = np.linalg.norm(host(M).astype(np.float64) - host(before).astype(np.float64), axis=0)
        th = np.degrees(2 * np.arcsin(np.minimum(1, ch / 2)))
        want = np.sort(th)[::-1][:dwg.top_count(n, frac)].mean()
        np.testing.assert_allclose(st[0, 1].item(), want, rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("n", [32_768, 32_769, 250_000, 1_000_000])
def test_equal_angles_over_repeated_iterations(n):
    """No weights: every angle is 0, in each of several iterations launched together."""
    from paper_2405_13839_amd import dwg
    P = cuda(np.random.default_rng(1).standard_normal((3, n)))
    N = cuda(unit_rows(np.random.default_rng(2), n))
    before = N.clone()
    _, st = dwg.iterate(P, torch.zeros(n, device="cuda"), None, N, dwg.Params(beta=2.3), max_iters=3, fixed_iters=True)
    assert st.shape == (3, 4) and not st[:, :3].any() and torch.equal(N, before)
