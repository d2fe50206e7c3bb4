"""Octree evaluation in segments of the node list, at the edges of the rule that counts them: one
segment of 64 sources, two and three of one source more, more segments than nodes, the most
there are; queries that end inside a wavefront and inside a run of blocks; nodes of one source."""
import numpy as np
import pytest

import oracle
from paper_2405_13839_amd import synth
from tests.helpers import TOL_G, TOL_W, cuda, e_g, e_w, host, unit_rows

pytestmark = pytest.mark.gpu


def _cloud(kind, n):
    if kind == "equal":  # one leaf at the deepest level: every segment but one is empty
        P = np.full((3, n), 0.25, np.float32)
        return P, np.full(n, 1.0 / n, np.float32)
    c = synth.torus_ellipsoids(max(n, 64), seed=n + 3)
    P = c.P[:, :n].copy()
    if kind == "copies":  # chains of cells and leaves of many sources
        P[:, n // 2:] = P[:, :1]
    return P, c.area[:n].copy()


CASES = [("torus", 1, 1, 16), ("torus", 64, 64, 16), ("torus", 65, 63, 4), ("torus", 129, 128, 1),
         ("torus", 4032, 65, 16), ("torus", 4097, 4097, 32), ("torus", 512, 512, 16), ("torus", 513, 65, 16), ("torus", 1025, 2049, 1),
         ("torus", 16_384, 257, 1), ("torus", 20_011, 2305, 16), ("copies", 3000, 700, 4), ("equal", 2000, 130, 16)]


@pytest.mark.parametrize("kind,n,m,leaf", CASES)
@pytest.mark.parametrize("lam", [0.0, 10.0])
def test_segments_match_the_oracle(kind, n, m, leaf, lam):
    from paper_2405_13839_amd import dwg
    P, area = _cloud(kind, n)
    rng = np.random.default_rng(n + m)
    N = unit_rows(rng, n)
    d = rng.uniform(0.02, 0.2, n).astype(np.float32)
    Q = rng.uniform(-1.5, 1.5, (3, m)).astype(np.float32)
    Q[:, :min(n, m) // 2] = P[:, :min(n, m) // 2]
    rw, rg, flag = oracle.tree_gwn(P, N, area, d, Q, lam=lam, beta=2.3, leaf=leaf)
    ok = flag == 0
    assert ok.mean() > 0.99
    args = [cuda(x) for x in (P, N, area, d, Q)]
    for comp in (True, False):
        prm = dwg.Params(lam=lam, beta=2.3, leaf=leaf, compensated=comp)
        w, g = dwg.gwn(*args, prm)
        assert e_w(host(w)[ok], rw[ok]) <= TOL_W and e_g(host(g)[:, ok], rg[:, ok]) <= TOL_G
        w1, _ = dwg.gwn(*args, prm, grad=False, want_wmean=True)
        assert e_w(host(w1)[ok], rw[ok]) <= TOL_W
    ws, gs = dwg.gwn_static(*args, dwg.Params(lam=lam, beta=2.3, leaf=leaf))
    assert e_w(host(ws)[ok], rw[ok]) <= TOL_W and e_g(host(gs)[:, ok], rg[:, ok]) <= TOL_G
