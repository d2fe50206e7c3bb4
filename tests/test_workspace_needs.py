"""dwg_workspace_bytes covers every call that its comment names, for sizes down to one point (no GPU: each call
is refused for a workspace of 64 bytes before any device access, and names the bytes that it needs)."""
import ctypes
import os
import random
import re

import pytest
import torch  # noqa: F401  (loads the HIP runtime libdwg links against)

from paper_2405_13839_amd import dwg

pytestmark = pytest.mark.skipif(not os.path.exists(dwg.LIB_PATH), reason="libdwg.so not built")
F = ctypes.c_void_p(0x1000)  # never dereferenced


def _needed(status):
    assert status == dwg.DWG_E_WORKSPACE, dwg.load().dwg_last_error()
    return int(re.search(r"(\d+) needed", dwg.load().dwg_last_error().decode()).group(1))


def _sizes():
    rng = random.Random(3)
    edges = [1, 2, 17, 18, 63, 64, 65, 127, 128, 129, 255, 256, 257, 512, 513, 4095, 4096, 4097, 8191, 8192, 16_384, 16_385,
             32_768, 32_769, 131_071, 131_072, 1 << 20, (1 << 20) + 1]
    for n in edges:
        for m in (1, 64, 129, 513, n, 200_000):
            yield n, m
    for _ in range(3000):
        yield int(10 ** rng.uniform(0, 7)), int(10 ** rng.uniform(0, 7))


@pytest.mark.parametrize("params", [None, dwg.Params(lam=4.0, split=5), dwg.Params(beta=2.3), dwg.Params(lam=1.0, beta=4.0, leaf=1),
                                    dwg.Params(beta=2.3, compensated=False)])
def test_field_calls(params):
    lib = dwg.load()
    kp = ctypes.byref(params.c()) if params else None
    ip = dwg.IterateParams(5, 0, 0.1, 0.01)
    out4, cnt = (ctypes.c_int64 * 4)(), ctypes.c_int64()
    for n, m in _sizes():
        size = dwg.workspace_bytes(n, m, params)
        assert _needed(lib.dwg_gwn_eval(F, F, F, None, n, F, m, kp, F, None, F, 64, None)) <= size, (n, m)
        assert _needed(lib.dwg_gwn_grad(F, F, F, None, n, F, m, kp, None, F, None, F, 64, None)) <= size, (n, m)
        own = dwg.workspace_bytes(n, n, params)
        assert _needed(lib.dwg_iterate(F, F, None, n, F, kp, ctypes.byref(ip), None, None, F, 64, None)) <= own, n
        if params and params.beta > 0:
            assert _needed(lib.dwg_octree_work(F, F, None, n, F, m, kp, out4, F, 64, None)) <= size, (n, m)
            assert _needed(lib.dwg_octree(F, n, params.leaf, F, F, 2 * n, ctypes.byref(cnt), F, 64, None)) <= own, n


def test_neighbour_and_network_calls():
    lib = dwg.load()
    for n, m in _sizes():
        size, own = dwg.workspace_bytes(n, m), dwg.workspace_bytes(n, n)
        k = min(16, n)
        assert _needed(lib.dwg_knn(F, n, F, m, 0, k, F, None, F, 64, None)) <= size, (n, m)
        assert _needed(lib.dwg_mlp_infer(F, F, n, F, F, 64, None)) <= own, n
        assert _needed(lib.dwg_mlp_train_step(F, F, F, 1, 1e-3, F, F, None, n, None, None, F, 64, None)) <= own, n
        if n < 18:
            continue
        assert _needed(lib.dwg_delta_knn_mean(F, n, 16, 1.0, F, F, 64, None)) <= own, n
        assert _needed(lib.dwg_delta_knn_window(F, n, 16, 0.0, 1.0, F, F, 64, None)) <= own, n
        assert _needed(lib.dwg_voronoi_area(F, n, 16, F, F, 64, None)) <= own, n
        for kind in (dwg.INIT_PCA, dwg.INIT_MLP):
            assert _needed(lib.dwg_init_normals(kind, ctypes.c_uint64(0), F, n, F, F, F, 64, None)) <= own, n
        for anchors in (17, 512, 4096):
            assert _needed(lib.dwg_delta_anchor_mean(F, n, 16, anchors, 1.0, F, F, 64, None)) <= own, n
            assert _needed(lib.dwg_features(F, n, anchors, F, F, 64, None)) <= own, n
