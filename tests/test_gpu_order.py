"""The radix sort behind the octree and the spatial order, at the sizes where it branches: one block
up to 4,096 elements, then tiles of 4,096 chained by look-back. The octree's permutation is the
stable order of the 63-bit cell codes, which NumPy gives exactly; the all-pairs path's own order
shows in the field only, which does not depend on it."""
import numpy as np
import pytest

import oracle
from paper_2405_13839_amd import synth
from tests.helpers import TOL_G, TOL_W, cuda, e_g, e_w, host, unit_rows

pytestmark = pytest.mark.gpu


def _codes(P):
    p = P.astype(np.float64)
    lo = p.min(1)
    ext = (p.max(1) - lo).max()
    sc = 2097152.0 / ext if ext > 0 else 0.0
    c = np.clip(np.floor((p - lo[:, None]) * sc), 0, 2097151).astype(np.uint64)
    code = np.zeros(P.shape[1], np.uint64)
    for b in range(21):
        for d in range(3):
            code |= ((c[d] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - d)
    return code


@pytest.mark.parametrize("kind", ["scene", "equal", "lattice"])
@pytest.mark.parametrize("n", [1, 65, 4095, 4096, 4097, 8193, 140_001])
def test_octree_permutation_is_the_stable_code_order(n, kind):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n)
    if kind == "scene":
        P = synth.torus_ellipsoids(max(n, 64), seed=3).P[:, :n].copy()
    elif kind == "equal":
        P = np.full((3, n), 0.25, np.float32)
    else:  # few distinct codes, so that ties decide
        P = (rng.integers(0, 5, (3, n)) / 4.0).astype(np.float32)
    perm, nodes = dwg.octree(cuda(P))
    np.testing.assert_array_equal(host(perm), np.argsort(_codes(P), kind="stable"))
    assert int(nodes[0, 0]) == 0 and int(nodes[0, 1]) == n


@pytest.mark.parametrize("n,m", [(4096, 4096), (4097, 4097), (4096, 4097), (9001, 300), (300, 9001)])
@pytest.mark.parametrize("lam", [0.0, 10.0])
def test_field_across_the_order_sizes(n, m, lam):
    from paper_2405_13839_amd import dwg
    c = synth.torus_ellipsoids(n, seed=n)
    rng = np.random.default_rng(m)
    N, d = unit_rows(rng, n), oracle.anchor_delta(c.P, n_anchor=256).astype(np.float32)
    Q = c.P if m == n else (c.P[:, rng.integers(0, n, m)] + rng.normal(0, 0.05, (3, m))).astype(np.float32)
    P = cuda(c.P)
    w, g = dwg.gwn(P, cuda(N), cuda(c.area), cuda(d), P if m == n else cuda(Q), dwg.Params(lam=lam))
    sel = np.unique(np.concatenate([np.arange(min(m, 64)), rng.integers(0, m, 64), [m - 1]]))
    rw, rg, flag = oracle.gwn(c.P, N, c.area, d, np.ascontiguousarray(Q[:, sel]), lam=lam)
    assert e_w(host(w)[sel], rw) <= TOL_W and e_g(host(g)[:, sel], rg, flag) <= TOL_G
