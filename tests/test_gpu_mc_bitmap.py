"""Grid cells and corners of the level set from bitmaps and from sorted codes: the number of cells on
both sides of the rule that chooses (the words of two bitmaps against the candidates), and the level
set itself with either way for cells and corners."""
import ctypes

import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

from oracle import mc
from paper_2405_13839_amd import synth
from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu


def _cells(P, depth, dilate):
    """Distinct cells of the points, grown by the rings, inside the cube."""
    x = P.astype(np.float64)
    lo = x.min(axis=1, keepdims=True)
    ext = float((x.max(axis=1, keepdims=True) - lo).max())
    c = np.clip(np.floor((x - lo) * (2097152.0 / ext)), 0, 2097151).astype(np.int64) >> (21 - depth)
    r = np.arange(-dilate, dilate + 1)
    off = np.stack(np.meshgrid(r, r, r), axis=-1).reshape(-1, 3)
    q = (c.T[:, None] + off[None]).reshape(-1, 3)
    q = q[((q >= 0) & (q < 1 << depth)).all(axis=1)]
    return len(np.unique(q, axis=0))


CASES = [(37, 5, 1), (38, 5, 1), (303, 6, 1), (304, 6, 1), (8191, 6, 0), (8192, 6, 0), (65, 6, 2), (66, 6, 2),
         (64, 1, 1), (64, 2, 1), (5000, 3, 2), (20_000, 8, 1), (3000, 9, 1), (50, 16, 1)]


@pytest.mark.parametrize("n,depth,dilate", CASES)
def test_number_of_cells(n, depth, dilate):
    from paper_2405_13839_amd import dwg
    lib = dwg.load()
    P = synth.torus_ellipsoids(max(n, 64), seed=n).P[:, :n].copy()
    Pc = cuda(P)
    mp = dwg.McParams(depth, dilate, 10, 0, 0)
    ws = torch.empty(int(lib.dwg_mc_workspace_bytes(n, ctypes.byref(dwg.Params().c()), ctypes.byref(mp), 0)),
                     dtype=torch.uint8, device="cuda")
    for _ in range(2):  # the second time over what the first left behind
        cells = ctypes.c_int64(0)
        st = lib.dwg_mc_cells(ctypes.c_void_p(Pc.data_ptr()), n, ctypes.byref(mp), ctypes.byref(cells),
                              ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0 and cells.value == _cells(P, depth, dilate)


@pytest.mark.parametrize("n,depth,dilate", [(120, 6, 1), (600, 6, 1), (2500, 5, 2), (2500, 6, 0), (400, 3, 1)])
def test_level_set_with_either(n, depth, dilate):
    from paper_2405_13839_amd import dwg
    s = synth.sphere(n, 0.002, 41)
    tri, iso = dwg.level_set(cuda(s.P), cuda(s.N_true), cuda(s.area), None, dwg.Params(), depth, dilate)
    tri = host(tri).astype(np.float64)
    otri, _, oiso, _, _ = mc.level_set(s.P, s.N_true, s.area, None, depth=depth, dilate=dilate)
    assert abs(iso - oiso) <= 1e-6
    assert abs(len(tri) - len(otri)) <= 0.002 * len(otri)
    d, _ = cKDTree(tri.mean(axis=1)).query(otri.mean(axis=1))
    assert np.mean(d < 1e-5) > 0.995
