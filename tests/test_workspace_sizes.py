"""Workspace sizes (no GPU): a size that was checked for a bound of the queries must hold what is laid
out for any smaller count, in both modes. The level-set update checks 8 cells + n queries and lays
out the distinct corners + n; a program may keep the workspace of its largest cloud for smaller ones."""
import ctypes
import os
import random

import pytest
import torch  # noqa: F401  (loads the HIP runtime libdwg links against)

from paper_2405_13839_amd import dwg

pytestmark = pytest.mark.skipif(not os.path.exists(dwg.LIB_PATH), reason="libdwg.so not built")

MODES = [dwg.Params(), dwg.Params(lam=10.0, split=7), dwg.Params(lam=10.0, beta=2.3), dwg.Params(beta=8.0, leaf=200)]


def _laid_out(params):
    """Bytes of the evaluation's layout for n sources and m queries (internal to the library)."""
    fn = dwg.load()["_ZN3dwg9gwn_bytesEllRK17dwg_kernel_paramsi"]
    fn.restype = ctypes.c_size_t
    fn.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(dwg.KernelParams), ctypes.c_int]
    kp = params.c()
    return lambda n, m: fn(n, m, ctypes.byref(kp), 0)


@pytest.mark.parametrize("params", MODES)
# noisy spheres with one ring around their cells: many points to a cell
@pytest.mark.parametrize("n,cells", [(200_000, 2_966), (300_000, 2_980), (400_000, 13_610), (500_000, 13_670),
                                     (1_000_000, 13_797), (2_000_000, 13_853), (2_000_000, 60_562),
                                     (133_604, 13_000), (56_835, 2_900), (1_030_000, 13_781)])
def test_level_set_layout_within_its_check(n, cells, params):
    size = _laid_out(params)
    bound = size(n, 8 * cells + n)
    for corners in sorted({8, cells, cells + cells // 3, 2 * cells, 4 * cells, 8 * cells}):
        for queries in (corners, corners + n):
            assert size(n, queries) <= bound, (corners, queries)


@pytest.mark.parametrize("params", MODES)
def test_layout_of_fewer_queries_or_sources_is_no_larger(params):
    size = _laid_out(params)
    rng = random.Random(1)
    for _ in range(40_000):
        n, m = int(10 ** rng.uniform(0, 7.3)), int(10 ** rng.uniform(0, 7.3))
        fewer = [max(1, int(v * rng.choice([1.0, 0.999, rng.random(), 10 ** -rng.uniform(0, 3)]))) for v in (n, m)]
        assert size(*fewer) <= size(n, m), (n, m, fewer)


@pytest.mark.parametrize("params", MODES)
def test_public_sizes_never_fall(params):
    """Step by step where the counts of splits change, and along a coarse sweep of everything."""
    steps = [512 * b + d for b in range(1, 700) for d in (-1, 0, 1)]
    steps += [64 * w for w in range(1900, 2300)] + [int(1.03 ** e) for e in range(120, 560)]
    last = 0
    for n in sorted(set(steps)):
        size = dwg.workspace_bytes(n, n, params)
        assert size >= last, n
        last = size
    kp, mp = params.c(), dwg.McParams(6, 1, 10, 0)
    last = 0
    for n in sorted({int(1.05 ** e) for e in range(150, 300)}):
        row = [dwg.load().dwg_mc_workspace_bytes(n, ctypes.byref(kp), ctypes.byref(mp), c)
               for c in (0, 1, 500, 2_966, 13_797, 13_853, 60_562, 10 ** 6)]
        assert row == sorted(row) and row[4] >= last, n
        last = row[4]


def test_room_for_the_partial_sums():
    """The room counted for partial sums holds splits x padded queries, also at the steps of the rules."""
    lib = dwg.load()
    fn = {}
    for name, args in (("choose_split", "lli"), ("split_columns", "lli"), ("tree_segments", "ll"), ("segment_columns", "ll")):
        f = lib[f"_ZN3dwg{len(name)}{name}E{args}"]
        f.argtypes = [ctypes.c_int64 if a == "l" else ctypes.c_int for a in args]
        f.restype = ctypes.c_int64 if name.endswith("columns") else ctypes.c_int
        fn[name] = f
    rng = random.Random(2)
    sizes = [int(10 ** rng.uniform(0, 9.3)) for _ in range(4000)]
    sizes += [64 * w + d for w in range(1, 4200, 7) for d in (-1, 0, 1)]
    for m in sizes:
        padded = -(-m // 512) * 512
        for n in (1, 63, 64, 65, 4096, 30_000, 1_000_000, m, int(10 ** rng.uniform(0, 9))):
            for split in (0, 0, 1, 5, 64):
                assert fn["split_columns"](n, m, split) >= fn["choose_split"](n, m, split) * padded, (n, m, split)
            assert fn["segment_columns"](n, m) >= fn["tree_segments"](n, m) * padded, (n, m)
