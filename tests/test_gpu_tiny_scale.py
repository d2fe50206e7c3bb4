"""Clouds so small that 1/r^3 of their shortest pairs overflows float32 (r below 1.4e-13): the guard for
coincident points bounds such pairs whichever loop a tile's distance would choose, so every sum is finite."""
import numpy as np
import pytest
import torch

from tests.helpers import cuda, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1366, 20_011])
@pytest.mark.parametrize("scale", [1e-12, 1e-13])
@pytest.mark.parametrize("compensated", [True, False])
def test_shortest_pairs_stay_finite(n, scale, compensated):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n)
    P = cuda(scale * rng.uniform(-1, 1, (3, n)))
    N = cuda(unit_rows(rng, n))
    area = torch.full((n,), 4 * scale * scale / n, device="cuda")
    prm = dwg.Params(compensated=compensated)
    w, g = dwg.gwn(P, N, area, None, P, prm)
    assert bool(torch.isfinite(w).all()) and bool(torch.isfinite(g).all())
    assert bool(torch.isfinite(dwg.gwn(P, N, area, None, P, prm, grad=False)).all())
