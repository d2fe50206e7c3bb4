"""The all-pairs field at the edges of its launches: single sources and queries, steps of 32 sources,
tiles of 256, blocks of 512 queries, the largest launch of the small kernel and the first beyond it;
with and without the gradient, split automatically and as asked."""
import numpy as np
import pytest

import oracle
from paper_2405_13839_amd import synth
from tests.helpers import TOL_G, TOL_W, cuda, e_g, e_w, host, unit_rows

pytestmark = pytest.mark.gpu

# 1,536 pairs of a query block and a tile: 48 x 32 and 49 x 32, 3 x 512 and 3 x 513
SIZES = [(1, 1), (31, 512), (32, 513), (33, 2), (255, 511), (256, 1), (257, 1025), (2000, 2000), (12_288, 16_384),
         (12_289, 16_384), (768, 262_144), (769, 262_144)]


@pytest.mark.parametrize("n,m", SIZES)
@pytest.mark.parametrize("lam", [0.0, 10.0])
def test_field_at_launch_edges(n, m, lam):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n * 7 + m)
    c = synth.torus_ellipsoids(max(n, 64), seed=n + 1)
    P, area, N = c.P[:, :n].copy(), c.area[:n].copy(), unit_rows(rng, n)
    d = rng.uniform(0.02, 0.3, n).astype(np.float32)
    Q = rng.uniform(-1.5, 1.5, (3, m)).astype(np.float32)
    Q[:, :min(n, m)] = P[:, :min(n, m)]
    sel = np.unique(np.concatenate([np.arange(min(m, 40)), rng.integers(0, m, 60), [m - 1]]))
    rw, rg, flag = oracle.gwn(P, N, area, d, np.ascontiguousarray(Q[:, sel]), lam=lam)
    args = [cuda(x) for x in (P, N, area, d, Q)]
    for prm in (dwg.Params(lam=lam), dwg.Params(lam=lam, compensated=False), dwg.Params(lam=lam, split=3),
                dwg.Params(lam=lam, split=64)):
        w, g = dwg.gwn(*args, prm)
        assert e_w(host(w)[sel], rw) <= TOL_W and e_g(host(g)[:, sel], rg, flag) <= TOL_G, prm
        w1, mean = dwg.gwn(*args, prm, grad=False, want_wmean=True)
        assert e_w(host(w1)[sel], rw) <= TOL_W, prm
        np.testing.assert_allclose(mean.item(), host(w1).astype(np.float64).mean(), rtol=1e-12, atol=1e-15)
