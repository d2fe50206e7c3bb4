"""Node sums, centres and opening radii at the sizes that change who forms them: 16 lanes up to 64
sources of a node, a wavefront up to 256, tiles of 256 and walks of 512 sources beyond. A wrong
centre, radius or moment of any node changes a far dipole or the choice to take it, so the field is
compared with the octree oracle's, at queries near and far, with kernel radii and without, and with
sources of no area."""
import numpy as np
import pytest

import oracle
from paper_2405_13839_amd import synth
from tests.helpers import TOL_G, TOL_W, cuda, e_g, e_w, host, unit_rows

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 16, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 4099, 33_333]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("leaf,radii", [(1, True), (16, False), (40, True), (16, True)])
def test_node_sums_at_their_edges(n, leaf, radii):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(31 * n + leaf)
    c = synth.torus_ellipsoids(max(n, 64), seed=n + leaf)
    pick = rng.permutation(c.n)[:n]
    P, area, N = c.P[:, pick].copy(), c.area[pick].copy(), unit_rows(rng, n)
    area[P[0] > 0.5] = 0.0
    area[0] = c.area[pick[0]]
    d = rng.uniform(0.01, 0.15, n).astype(np.float32) if radii else None
    m = 500
    Q = rng.uniform(-3.0, 3.0, (3, m)).astype(np.float32)
    Q[:, :250] = P[:, rng.integers(0, n, 250)] + rng.normal(0, 0.05, (3, 250)).astype(np.float32)
    rw, rg, flag = oracle.tree_gwn(P, N, area, d, Q, lam=0.0, beta=2.0, leaf=leaf)
    ok = flag == 0
    assert ok.mean() > 0.99
    w, g = dwg.gwn(cuda(P), cuda(N), cuda(area), None if d is None else cuda(d), cuda(Q),
                   dwg.Params(beta=2.0, leaf=leaf))
    assert e_w(host(w)[ok], rw[ok]) <= TOL_W and e_g(host(g)[:, ok], rg[:, ok]) <= TOL_G
