"""The level-set update for the neighbour counts at the ends of their range and one that divides no
wavefront: every face's vector reaches its k nearest points, component by component."""
import numpy as np
import pytest

import oracle
from oracle import mc
from paper_2405_13839_amd import synth
from tests.helpers import angle_deg, cuda, host, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 3, 16])
@pytest.mark.parametrize("surface", ["cubes", "tets"])
def test_every_neighbour_receives_its_faces(k, surface):
    from paper_2405_13839_amd import dwg
    c = synth.torus_ellipsoids(2500, seed=4300 + k)
    N0 = unit_rows(np.random.default_rng(k), c.n)
    d = oracle.anchor_delta(c.P).astype(np.float32)
    Nt = cuda(N0)
    _, stats = dwg.iterate_mc(cuda(c.P), cuda(c.area), cuda(d), Nt, dwg.Params(lam=10.0), depth=5, dilate=1, k=k,
                              max_iters=1, fixed_iters=True, surface=surface)
    N1, oiso, _, cnt = mc.update(c.P, N0, c.area, d, lam=10.0, depth=5, dilate=1, k=k, beta=0.0, surface=surface)
    assert abs(stats[0, 0].item() - oiso) <= 1e-5
    ang = angle_deg(host(Nt), N1)
    assert np.mean(ang <= 0.1) > 0.99 and np.median(ang) <= 1e-3
    keep = cnt == 0
    if keep.any():
        assert np.all(angle_deg(host(Nt)[:, keep], N0[:, keep]) < 1e-4)
