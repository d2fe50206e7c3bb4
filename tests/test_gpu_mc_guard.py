"""The level-set entry points write nothing past a workspace of exactly the stated size: clouds with
many points to a grid cell, where the queries there are and the bound that the size is for lie on
either side of a step in the number of source splits or octree segments."""
import ctypes

import numpy as np
import pytest
import torch

from tests.helpers import cuda, unit_rows

pytestmark = pytest.mark.gpu
GUARD = 96 << 20


@pytest.mark.parametrize("n,depth,beta", [(1_000_000, 5, 2.3), (300_000, 4, 2.3), (133_604, 5, 2.3), (56_835, 4, 0.0)])
@pytest.mark.parametrize("iso", ["points", "corners"])
def test_nothing_written_past_the_workspace(n, depth, beta, iso):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n)
    u = unit_rows(rng, n)
    P = cuda(u + 0.005 * rng.standard_normal((3, n)))
    area = torch.full((n,), 4 * np.pi / n, device="cuda")
    prm = dwg.Params(lam=10.0, beta=beta)
    size = dwg.mc_workspace(P, prm, depth, iso=iso).numel()
    buf = torch.full((size + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    N = cuda(u)
    dwg.iterate_mc(P, area, None, N, prm, depth=depth, max_iters=1, fixed_iters=True, ws=buf[:size], iso=iso)
    tri, w_bar = dwg.level_set(P, N, area, None, prm, depth=depth, ws=buf[:size], iso=iso)
    assert bool((buf[size:] == 0xA5).all())
    # both ran in full: w_bar lies between the outside's 0 and the inside's 1, the surface is the sphere's
    assert 0.0 < w_bar < 1.0 and tri.shape[0] > 1000
    assert abs(float(tri.norm(dim=2).mean()) - 1.0) < 2.0 ** (1 - depth)
    # and gives bit for bit what it gives with room to spare
    N1 = cuda(u)
    dwg.iterate_mc(P, area, None, N1, prm, depth=depth, max_iters=1, fixed_iters=True, ws=buf, iso=iso)
    assert torch.equal(N, N1) and not torch.equal(N, cuda(u))
    # a byte less is refused
    mp, kp = dwg.McParams(depth, 1, 10, 0 if iso == "points" else 1, 0), prm.c()
    st = dwg.load().dwg_level_set(*(ctypes.c_void_p(t.data_ptr()) for t in (P, N, area)), None, n, ctypes.byref(kp),
                                  ctypes.byref(mp), ctypes.c_void_p(tri.data_ptr()), tri.shape[0],
                                  ctypes.byref(ctypes.c_int64()), ctypes.byref(ctypes.c_double()),
                                  ctypes.c_void_p(buf.data_ptr()), size - 1, None)
    assert st == dwg.DWG_E_WORKSPACE
