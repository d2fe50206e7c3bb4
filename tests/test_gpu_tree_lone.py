"""Octree evaluation with one wavefront per block (131,072 queries and more) and with four: both sides
of the rule, with a last block that is not full, give the oracle's field at sampled queries."""
import numpy as np
import pytest
import torch

import oracle
from paper_2405_13839_amd import synth
from tests.helpers import TOL_G, TOL_W, cuda, e_g, e_w, host, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [131_071, 131_072, 131_137])
@pytest.mark.parametrize("grad", [True, False])
def test_blocks_of_one_and_four_wavefronts(m, grad):
    from paper_2405_13839_amd import dwg
    c = synth.torus_ellipsoids(3000, seed=77)
    rng = np.random.default_rng(5)
    N = unit_rows(rng, c.n)
    d = rng.uniform(0.02, 0.2, c.n).astype(np.float32)
    Q = rng.uniform(-1.5, 1.5, (3, 131_137)).astype(np.float32)[:, :m].copy()
    prm = dwg.Params(lam=10.0, beta=2.3)
    out = dwg.gwn(*[cuda(x) for x in (c.P, N, c.area, d, Q)], prm, grad=grad)
    w = host(out[0] if grad else out)
    sel = np.unique(np.concatenate([rng.integers(0, m, 300), np.arange(m - 130, m)]))
    rw, rg, flag = oracle.tree_gwn(c.P, N, c.area, d, np.ascontiguousarray(Q[:, sel]), lam=10.0, beta=2.3, leaf=32)
    ok = flag == 0
    assert ok.mean() > 0.99 and e_w(w[sel][ok], rw[ok]) <= TOL_W
    if grad:
        assert e_g(host(out[1])[:, sel][:, ok], rg[:, ok]) <= TOL_G
    torch.cuda.synchronize()
