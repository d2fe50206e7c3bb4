"""Performance cases of the framework: what a program that orients point clouds has it do.

Every case goes through the public functions of paper_2405_13839_amd.dwg on inputs that are
drawn on the GPU from a seed. The scene is the benchmark's family (a torus united with two
ellipsoids, 5% uniform outliers, noise 0.25% of the diagonal), or the noisy unit sphere of the
smallest workload. `listed()` holds the named sizes, `draw()` gives more of the same kinds.

Kinds
  iterate  DWG iterations with every point as a query: all pairs (beta = 0) or octree (beta > 0)
  field    w, or w and its gradient, of an oriented cloud at queries (its own points or others)
  radius   the anchor kernel radius, first stage of every solve
  learned  the learned initial normals: anchor features and the MLP forward pass
  areas    Voronoi area weights and the windowed kernel radius of an unweighted scan
  knn      nearest neighbours (indices and distances)
  train    one optimiser step of the MLP: forward, backward, Adam
  update   iterations of the level-set update on a grid of 2^depth cells per axis
"""
import math
import os

import numpy as np
import torch

from paper_2405_13839_amd import dwg, mlp_init

DEV = "cuda"
FOUR_PI = 4.0 * math.pi
ANCHORS = 4096
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(dwg.__file__)), "weights", "mlp_init.safetensors")


def listed():
    return [
        # the smallest solve: 2,000 points of a sphere, plain kernel, a few iterations per call
        {"name": "iterate_2k", "kind": "iterate", "shape": "sphere", "n": 2000, "lam": 0.0, "beta": 0.0, "iters": 4},
        # the 100K-point scene evaluated exactly at its own points
        {"name": "field_100k", "kind": "field", "shape": "scene", "n": 100_000, "m": 0, "lam": 10.0, "beta": 0.0,
         "grad": True},
        # inside/outside values of a plain field at other queries: no gradient, ragged sizes
        {"name": "inside_131k", "kind": "field", "shape": "scene", "n": 49_999, "m": 131_075, "lam": 0.0, "beta": 0.0,
         "grad": False},
        # one exact iteration of the 1M-point scene: the benchmark's step
        {"name": "iterate_1m", "kind": "iterate", "shape": "scene", "n": 1_000_000, "lam": 10.0, "beta": 0.0,
         "iters": 1},
        # octree solve of the 1M-point scene, in slices of four iterations
        {"name": "octree_1m", "kind": "iterate", "shape": "scene", "n": 1_000_000, "lam": 10.0, "beta": 2.3,
         "iters": 4},
        # octree solve of a small scan
        {"name": "octree_20k", "kind": "iterate", "shape": "scene", "n": 20_011, "lam": 4.0, "beta": 2.3, "iters": 4},
        # kernel radius of the 1M-point scene
        {"name": "radius_1m", "kind": "radius", "shape": "scene", "n": 1_000_000, "k": 10},
        # learned initial normals of the 1M-point scene
        {"name": "learned_1m", "kind": "learned", "shape": "scene", "n": 1_000_000},
        # a scan without weights: Voronoi areas of 15 neighbours, radius of 10
        {"name": "areas_131k", "kind": "areas", "shape": "scene", "n": 131_071},
        # neighbours of a small cloud's own points
        {"name": "knn_50k", "kind": "knn", "shape": "scene", "n": 50_001, "m": 0, "k": 10},
        # a step of the training run: batches of 8,192 rows, outliers masked out
        {"name": "train_8192", "kind": "train", "rows": 8192, "step": 100},
        # the level-set update of a 100K-point scene, octree evaluation on a grid of depth 7
        {"name": "update_100k", "kind": "update", "shape": "scene", "n": 100_000, "lam": 10.0, "beta": 2.3,
         "depth": 7, "iters": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["iterate", "iterate", "field", "field", "radius", "learned", "areas", "knn", "train",
                       "update"])
    shape = rng.choice(["scene", "scene", "sphere"])
    lam = rng.choice([0.0, 4.0, 10.0, 50.0])
    if kind == "iterate":
        beta = rng.choice([0.0, 2.3, 2.3, 8.0])
        n = _log(rng, 1000, 200_000) if beta == 0.0 else _log(rng, 1000, 1_000_000 if beta < 8.0 else 400_000)
        return {"kind": kind, "shape": shape, "n": n, "lam": lam, "beta": beta, "iters": rng.randint(1, 4)}
    if kind == "field":
        beta = rng.choice([0.0, 0.0, 2.3])
        n, m = _log(rng, 500, 150_000), rng.choice([0, _log(rng, 200, 200_000)])
        return {"kind": kind, "shape": shape, "n": n, "m": m, "lam": lam, "beta": beta,
                "grad": rng.choice([True, True, False])}
    if kind == "radius":
        return {"kind": kind, "shape": shape, "n": _log(rng, 5000, 1_000_000), "k": rng.randint(6, 16)}
    if kind == "learned":
        return {"kind": kind, "shape": shape, "n": _log(rng, 5000, 1_000_000)}
    if kind == "areas":
        return {"kind": kind, "shape": shape, "n": _log(rng, 1000, 1_000_000)}
    if kind == "knn":
        return {"kind": kind, "shape": shape, "n": _log(rng, 1000, 500_000),
                "m": rng.choice([0, _log(rng, 500, 300_000)]), "k": rng.randint(1, 16)}
    if kind == "train":
        return {"kind": kind, "rows": _log(rng, 64, 65_536), "step": rng.randint(20, 1000)}
    return {"kind": kind, "shape": shape, "n": _log(rng, 5000, 200_000), "lam": lam, "beta": 2.3,
            "depth": rng.randint(5, 8), "iters": rng.randint(1, 3)}


# ------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(DEV)
    g.manual_seed(seed)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _unit(x):
    return x / x.norm(dim=0, keepdim=True).clamp_min(1e-300)


def _torus(g, m):
    """m points by area on the torus R = 1, r = 0.3, with their outward normals: [3, m] each."""
    k = 2 * m + 64
    th, ph = 2 * math.pi * _rand(g, k), 2 * math.pi * _rand(g, k)
    keep = _rand(g, k) < (1.0 + 0.3 * torch.cos(th)) / 1.3
    th, ph = th[keep][:m], ph[keep][:m]
    nv = torch.stack([torch.cos(th) * torch.cos(ph), torch.cos(th) * torch.sin(ph), torch.sin(th)])
    ring = torch.stack([torch.cos(ph), torch.sin(ph), torch.zeros_like(ph)])
    return ring + 0.3 * nv, nv


def _ellipsoid(g, m, ax, rot, centre):
    a, b, c = ax
    k = 4 * m + 64
    u = _unit(_randn(g, 3, k))
    wgt = torch.sqrt((b * c * u[0]) ** 2 + (a * c * u[1]) ** 2 + (a * b * u[2]) ** 2)
    u = u[:, _rand(g, k) < wgt / max(b * c, a * c, a * b)][:, :m]
    axt = torch.tensor(ax, device=DEV, dtype=torch.float64)[:, None]
    return rot @ (u * axt) + centre, _unit(rot @ (u / axt))


def _ellipsoid_area(ax):
    """Knud Thomsen's formula (within 1.1%)."""
    a, b, c = (v ** 1.6075 for v in ax)
    return FOUR_PI * ((a * b + a * c + b * c) / 3.0) ** (1 / 1.6075)


def _cloud(shape, n, seed):
    """(P [3, n] float32, area [n] float32, outward normals [3, n] float64, 0 for outliers)."""
    g = _gen(seed)
    if shape == "sphere":
        u = _unit(_randn(g, 3, n))
        p = u + 0.005 * _randn(g, 3, n)
        return p.float().contiguous(), torch.full((n,), FOUR_PI / n, device=DEV), u
    r = np.random.Generator(np.random.PCG64(seed))
    parts, areas = [], [4 * math.pi ** 2 * 0.3]
    for _ in range(2):
        ax = [float(v) for v in r.uniform(0.2, 0.6, 3)]
        centre = torch.tensor([r.uniform(-1.3, 1.3), r.uniform(-1.3, 1.3), r.uniform(-0.5, 0.5)], device=DEV)[:, None]
        q, _ = np.linalg.qr(r.standard_normal((3, 3)))
        parts.append((ax, torch.from_numpy(q).to(DEV), centre.double()))
        areas.append(_ellipsoid_area(ax))
    n_out = n // 20
    n_in, over = n - n_out, 1.4
    while True:
        xs, ns, seen = [], [], 0.0
        for k in range(3):
            m = int(over * n_in * areas[k] / sum(areas)) + 64
            x, nv = _torus(g, m) if k == 0 else _ellipsoid(g, m, *parts[k - 1])
            out = torch.ones(x.shape[1], dtype=torch.bool, device=DEV)
            if k > 0:
                out &= (torch.sqrt(x[0] ** 2 + x[1] ** 2) - 1.0) ** 2 + x[2] ** 2 >= 0.09
            for j, (ax, rot, centre) in enumerate(parts):
                if j + 1 != k:
                    y = (rot.T @ (x - centre)) / torch.tensor(ax, device=DEV, dtype=torch.float64)[:, None]
                    out &= (y * y).sum(0) >= 1.0
            seen += areas[k] * float(out.double().mean())
            xs.append(x[:, out])
            ns.append(nv[:, out])
        x, nv = torch.cat(xs, 1), torch.cat(ns, 1)
        if x.shape[1] >= n_in:
            break
        over *= 1.5
    sel = torch.randperm(x.shape[1], generator=g, device=DEV)[:n_in]
    x, nv = x[:, sel], nv[:, sel]
    lo, hi = x.amin(1, keepdim=True), x.amax(1, keepdim=True)
    x = x + 0.0025 * (hi - lo).norm() * _randn(g, 3, n_in)
    p = torch.cat([x, lo + (hi - lo) * _rand(g, 3, n_out)], 1)
    nv = torch.cat([nv, torch.zeros(3, n_out, device=DEV, dtype=torch.float64)], 1)
    perm = torch.randperm(n, generator=g, device=DEV)
    return p[:, perm].float().contiguous(), torch.full((n,), seen / n_in, device=DEV), nv[:, perm]


def _near(P, A, k, skip=None):
    """Distances (float64, ascending) and indices of the k nearest columns of A for each column
    of P; skip[i] is left out for point i (-1: none)."""
    n, d_out, i_out = P.shape[1], [], []
    rows = max(1, min(n, (1 << 28) // A.shape[1]))
    for s in range(0, n, rows):
        p = P[:, s:s + rows].double()
        d2 = sum((p[c][:, None] - A[c].double()[None, :]) ** 2 for c in range(3))
        if skip is not None:
            j = skip[s:s + rows]
            at = torch.nonzero(j >= 0)[:, 0]
            d2[at, j[at]] = math.inf
        v, i = torch.topk(d2, k, dim=1, largest=False, sorted=True)
        d_out.append(v.sqrt())
        i_out.append(i)
    return torch.cat(d_out), torch.cat(i_out)


def _anchors(P, count=ANCHORS):
    """Anchor points (every stride-th) and each point's own anchor (-1: it is none)."""
    n = P.shape[1]
    stride = max(1, n // count)
    i = torch.arange(n, device=DEV)
    return P[:, ::stride].contiguous(), torch.where(i % stride == 0, i // stride, -1)


def _radius(P, k=10):
    A, own = _anchors(P)
    return _near(P, A, k, own)[0].mean(1)


def _normals(nv, seed, spread=0.6):
    """The normals with the error that the learned initialisation has (34 degrees on average);
    uniform at the outliers."""
    return _unit(nv + spread * _randn(_gen(seed + 77_777), *nv.shape)).float().contiguous()


def _queries(P, m, seed):
    """m queries in the cloud's box grown by a tenth on each side."""
    lo, hi = P.amin(1, keepdim=True).double(), P.amax(1, keepdim=True).double()
    return (lo + (hi - lo) * (1.2 * _rand(_gen(seed + 55_555), 3, m) - 0.1)).float().contiguous()


def _features(P, at=None):
    """Anchor features [rows, 48] (float64) of the points `at` (default: all)."""
    A, own = _anchors(P)
    if at is not None:
        P, own = P[:, at], own[at]
    dist, idx = _near(P, A, 16, own)
    x = (A.double().T[idx] - P.double().T[:, None]) / dist.mean(1)[:, None, None]
    return x.reshape(-1, 48)


def _train_state(rows, seed):
    """A batch drawn from a training scene (features, analytic normals, outliers masked out) and
    the state of a run in its first steps (moments of the size that its gradients have)."""
    P, _, nv = _cloud("scene", max(50_000, rows), seed)
    g = _gen(seed + 33_333)
    at = torch.randperm(P.shape[1], generator=g, device=DEV)[:rows]
    count = mlp_init.N_PARAMS
    return {
        "params": torch.from_numpy(mlp_init.init_params(seed)).to(DEV),
        "m": (1e-3 * _randn(g, count)).float(),
        "v": ((2e-3 * (0.5 + _rand(g, count))) ** 2).float(),
        "X": _features(P, at).float().contiguous(),
        "T": nv[:, at].T.float().contiguous(),
        "mask": (nv[:, at].norm(dim=0) > 0.5).to(torch.uint8),
    }


def _params(case):
    return dwg.Params(lam=case["lam"], beta=case["beta"])


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind == "train":
        s.update(_train_state(case["rows"], seed))
        return s
    P, area, nv = _cloud(case["shape"], case["n"], seed)
    n = P.shape[1]
    s["P"] = P
    if kind in ("iterate", "field", "update"):
        s["area"], s["delta"], s["N"] = area, _radius(P).float(), _normals(nv, seed)
        s["params"] = _params(case)
    if kind == "iterate":
        s["ws"] = dwg.workspace(n, n, P.device, s["params"])
    elif kind == "field":
        s["Q"] = _queries(P, case["m"], seed) if case["m"] else P
        s["ws"] = dwg.workspace(n, s["Q"].shape[1], P.device, s["params"])
    elif kind == "update":
        s["ws"] = dwg.mc_workspace(P, s["params"], case["depth"])
    elif kind == "knn":
        s["Q"] = _queries(P, case["m"], seed) if case["m"] else P
        s["ws"] = dwg.workspace(n, s["Q"].shape[1], P.device)
    else:
        s["ws"] = dwg.workspace(n, n, P.device)
        if kind == "areas":
            s["side"] = float((P.amax(1) - P.amin(1)).max())
        if kind == "learned":
            s["mlp"] = mlp_init.load_params(WEIGHTS, DEV)
    return s


def _stats(st):
    """Per iteration w_bar, the convergence statistic and the mean chord (the fourth column is
    a duration)."""
    return [[float(v) for v in row[:3]] for row in st]


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "iterate":
        N = s["N"].clone()
        status, st = dwg.iterate(s["P"], s["area"], s["delta"], N, s["params"], max_iters=case["iters"],
                                 fixed_iters=True, ws=s["ws"])
        return {"N": N, "status": status, "stats": _stats(st)}
    if kind == "field":
        got = dwg.gwn(s["P"], s["N"], s["area"], s["delta"], s["Q"], s["params"], grad=case["grad"], ws=s["ws"])
        return {"w": got[0], "grad": got[1]} if case["grad"] else {"w": got}
    if kind == "radius":
        return {"delta": dwg.delta_anchor_mean(s["P"], case["k"], ANCHORS, 1.0, ws=s["ws"])}
    if kind == "learned":
        return {"N": dwg.mlp_normals(s["P"], s["mlp"], ws=s["ws"])}
    if kind == "areas":
        area = dwg.voronoi_area(s["P"], 15, ws=s["ws"])
        return {"area": area, "delta": dwg.delta_knn_window(s["P"], 10, 0.0015 * s["side"], 0.015 * s["side"],
                                                            ws=s["ws"])}
    if kind == "knn":
        idx, dist = dwg.knn(s["P"], s["Q"], case["k"], self_skip=case["m"] == 0, ws=s["ws"])
        return {"idx": idx, "dist": dist}
    if kind == "train":
        loss, grad = dwg.mlp_train_step(s["params"], s["m"], s["v"], case["step"], 1e-3, s["X"], s["T"], s["mask"],
                                        want_grad=True)
        return {"params": s["params"], "m": s["m"], "v": s["v"], "loss": loss, "grad": grad}
    N = s["N"].clone()
    status, st = dwg.iterate_mc(s["P"], s["area"], s["delta"], N, s["params"], depth=case["depth"],
                                max_iters=case["iters"], fixed_iters=True, ws=s["ws"])
    return {"N": N, "status": status, "stats": _stats(st)}


# --------------------------------------------------------------------------------- work
def _interactions(n, beta):
    """Far dipoles and leaf pairs per query of the octree traversal with leaves of 32 sources, as
    dwg.octree_work counts them on the scene (within a third from 5,000 to 1M points)."""
    return min(float(n), (60.0 * (n / 1000.0) ** 0.36 + 140.0 + 0.0024 * n) * (beta / 2.3) ** 1.4)


def work(case):
    kind = case["kind"]
    if kind == "train":
        b, par = case["rows"], mlp_init.N_PARAMS
        return {"bytes": b * (48 + 3) * 4 + b + par * 4 * 7, "flops": 3.0 * 2 * (48 * 128 + 128 * 128 + 128 * 3) * b}
    n = case["n"]
    if kind in ("iterate", "field"):
        m = n if kind == "iterate" else (case["m"] or n)
        grad = kind == "iterate" or case["grad"]
        fl = (44 if grad else 24) if case["lam"] > 0 else (32 if grad else 18)
        per = n if case["beta"] == 0.0 else _interactions(n, case["beta"])
        its = case.get("iters", 1)
        return {"bytes": its * (32 * n + 12 * m + (16 if grad else 4) * m), "flops": float(its) * fl * per * m}
    if kind == "radius":
        return {"bytes": 16 * n, "flops": 0}
    if kind == "learned":
        return {"bytes": 24 * n, "flops": 2.0 * (48 * 128 + 128 * 128 + 128 * 3) * n}
    if kind == "areas":
        return {"bytes": 2 * 16 * n, "flops": 0}
    if kind == "knn":
        m = case["m"] or n
        return {"bytes": 12 * n + 12 * m + 8 * case["k"] * m, "flops": 0}
    corners = min(6.0 * n, 1.6 * 4 ** case["depth"])  # of the cells that hold points and their neighbours
    fl = (24 if case["lam"] > 0 else 18) * _interactions(n, case["beta"])
    return {"bytes": case["iters"] * (44 * n + 20 * corners), "flops": case["iters"] * fl * (corners + n)}


# -------------------------------------------------------------------- values in 64 bits
def _pair_sums(d, nrm, a, dl, lam):
    """w and gradient terms of pairs: d [3, ...] source minus query, normals [3, ...], areas,
    radii (0: none)."""
    r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
    r, s = r2.sqrt(), math.sqrt(lam)
    rho = torch.maximum(r, dl)
    f = torch.where(r2 > 0, a * torch.exp(-s * r) / (FOUR_PI * rho ** 3), 0.0)
    phi = f * (1 + s * r)
    c = d[0] * nrm[0] + d[1] * nrm[1] + d[2] * nrm[2]
    t = c * (torch.where((rho == r) & (r2 > 0), 3 * phi / r2.clamp_min(1e-300), 0.0) + f * lam)
    return c * phi, phi, t


def _all_pairs(P, N, a, dl, Q, lam):
    P, N, a, dl, Q = (x.double() for x in (P, N, a, dl, Q))
    n, m = P.shape[1], Q.shape[1]
    w, g = torch.empty(m, device=DEV, dtype=torch.float64), torch.empty(3, m, device=DEV, dtype=torch.float64)
    rows = max(1, (1 << 26) // n)
    for s in range(0, m, rows):
        q = Q[:, s:s + rows]
        d = [P[c][None, :] - q[c][:, None] for c in range(3)]
        wt, phi, t = _pair_sums(d, [N[c][None, :] for c in range(3)], a[None, :], dl[None, :], lam)
        w[s:s + rows] = wt.sum(1)
        for c in range(3):
            g[c, s:s + rows] = (t * d[c]).sum(1) - phi @ N[c]
    return w, g


class _Octree:
    """The octree of the sources, level by level (21 levels of the cube over their box)."""

    def __init__(self, P, a, dl, beta, leaf=32):
        p = P.double()
        n = p.shape[1]
        lo = p.amin(1)
        side = (p.amax(1) - lo).max()
        cell = torch.floor((p - lo[:, None]) * (2097152.0 / side)).clamp(0, 2097151).long()
        code = torch.zeros(n, dtype=torch.long, device=DEV)
        for b in range(21):
            for c in range(3):
                code |= ((cell[c] >> b) & 1) << (3 * b + 2 - c)
        code, self.perm = torch.sort(code, stable=True)
        self.p, self.a, self.dl = p[:, self.perm], a.double()[self.perm], dl.double()[self.perm]
        self.levels = []
        start, end = torch.zeros(1, dtype=torch.long, device=DEV), torch.full((1,), n, device=DEV)
        cum = torch.cat([torch.zeros(4, 1, device=DEV, dtype=torch.float64),
                         torch.cumsum(torch.cat([self.a[None], self.a * self.p]), 1)], 1)
        for level in range(22):
            size = end - start
            node = torch.repeat_interleave(torch.arange(len(start), device=DEV), size)
            src = self._expand(start, size)
            tot = cum[:, end] - cum[:, start]
            cen = tot[1:] / tot[0]
            zero = torch.zeros(len(start), device=DEV, dtype=torch.float64)
            r = zero.scatter_reduce(0, node, (self.p[:, src] - cen[:, node]).norm(dim=0), "amax")
            dm = zero.scatter_reduce(0, node, self.dl[src], "amax")
            is_leaf = (size <= leaf) | (level == 21)
            lv = {"start": start, "size": size, "cen": cen, "crit2": torch.maximum(beta * r, r + dm) ** 2,
                  "leaf": is_leaf}
            self.levels.append(lv)
            if bool(is_leaf.all()):
                break
            key = code >> (3 * (20 - level))
            head = torch.ones(n, dtype=torch.bool, device=DEV)
            head[1:] = key[1:] != key[:-1]
            keep = ~is_leaf[node]
            at = src[keep]
            first = head[at]
            first[0] = True
            par = node[keep]
            first[1:] |= par[1:] != par[:-1]
            begin = torch.nonzero(first)[:, 0]
            start, par = at[begin], par[begin]
            end = start + torch.diff(begin, append=torch.tensor([len(at)], device=DEV))
            kids = torch.bincount(par, minlength=len(size))
            lv["kids"], lv["first"] = kids, torch.cumsum(kids, 0) - kids

    @staticmethod
    def _expand(start, count):
        base = torch.cumsum(count, 0) - count
        return torch.arange(int(count.sum()), device=DEV) + torch.repeat_interleave(start - base, count)

    def field(self, N, Q, lam):
        nrm = N.double()[:, self.perm]
        cum = torch.cat([torch.zeros(3, 1, device=DEV, dtype=torch.float64), torch.cumsum(self.a * nrm, 1)], 1)
        m = Q.shape[1]
        w, g = torch.zeros(m, device=DEV, dtype=torch.float64), torch.zeros(3, m, device=DEV, dtype=torch.float64)
        for s in range(0, m, 4096):
            q = Q[:, s:s + 4096].double()
            qi = torch.arange(q.shape[1], device=DEV)
            node = torch.zeros_like(qi)
            for lv in self.levels:
                d = lv["cen"][:, node] - q[:, qi]
                far = (d ** 2).sum(0) > lv["crit2"][node]
                lf = lv["leaf"][node] & ~far
                f, j = torch.nonzero(far)[:, 0], node[far]
                mom = cum[:, lv["start"][j] + lv["size"][j]] - cum[:, lv["start"][j]]
                one = torch.ones(len(f), device=DEV, dtype=torch.float64)
                self._add(w, g, s + qi[f], d[:, f], mom, one, 0 * one, lam)
                count = lv["size"][node[lf]]
                src = self._expand(lv["start"][node[lf]], count)
                ql = torch.repeat_interleave(qi[lf], count)
                self._add(w, g, s + ql, self.p[:, src] - q[:, ql], nrm[:, src], self.a[src], self.dl[src], lam)
                go = ~far & ~lf
                if not bool(go.any()):
                    break
                kids = lv["kids"][node[go]]
                node, qi = self._expand(lv["first"][node[go]], kids), torch.repeat_interleave(qi[go], kids)
        return w, g

    @staticmethod
    def _add(w, g, at, d, nrm, a, dl, lam):
        wt, phi, t = _pair_sums(d, nrm, a, dl, lam)
        w.index_add_(0, at, wt)
        g.index_add_(1, at, t * d - phi * nrm)


def _mlp64(prm, x):
    """The MLP's output before normalisation; prm a flat float64 blob."""
    o = 0
    for k, (_, shp) in enumerate(mlp_init.SHAPES):
        cnt = math.prod(shp)
        v = prm[o:o + cnt].reshape(shp)
        x = x @ v.T if len(shp) == 2 else (torch.relu(x + v) if k < 5 else x + v)
        o += cnt
    return x


def _voronoi64(P, idx):
    """Area of each point's cell in the Voronoi diagram of its neighbours' projections: a square
    of the largest projected distance cut by the bisectors, as a sum over its edges."""
    p = P.double().T
    nb = p[idx]
    x = torch.cat([p[:, None], nb], 1)
    x = x - x.mean(1, keepdim=True)
    cov = (x.transpose(1, 2).contiguous() @ x).cpu()
    nv = torch.linalg.eigh(cov)[1][:, :, 0].to(DEV)
    e = torch.zeros_like(nv).scatter_(1, nv.abs().argmin(1, keepdim=True), 1.0)
    u = torch.linalg.cross(nv, e)
    u = u / u.norm(dim=1, keepdim=True)
    v = torch.linalg.cross(nv, u)
    d = nb - p[:, None]
    q = torch.stack([(d * u[:, None]).sum(2), (d * v[:, None]).sum(2)], 2)
    big = q.norm(dim=2).amax(1)
    box = torch.tensor([[1.0, 0.0], [-1.0, 0.0], [0.0, 1.0], [0.0, -1.0]], device=DEV, dtype=torch.float64)
    nrm = torch.cat([q, box.expand(len(p), 4, 2)], 1)
    b = torch.cat([0.5 * (q ** 2).sum(2), big[:, None].expand(-1, 4)], 1)
    twice = torch.zeros(len(p), device=DEV, dtype=torch.float64)
    for t in range(nrm.shape[1]):
        a, bt = nrm[:, t], b[:, t]
        foot = a * (bt / (a ** 2).sum(1))[:, None]
        den = nrm[:, :, 1] * a[:, None, 0] - nrm[:, :, 0] * a[:, None, 1]
        num = b - (nrm * foot[:, None]).sum(2)
        other = torch.arange(nrm.shape[1], device=DEV) != t
        hi = torch.where((den > 0) & other, num / den, math.inf).amin(1)
        low = torch.where((den < 0) & other, num / den, -math.inf).amax(1)
        twice += torch.where((hi > low) & (bt > 0), bt * (hi - low), 0.0)
    return 0.5 * twice


def _iterate64(s, case, field):
    N = s["N"].double()
    stats = []
    top = max(1, math.ceil(0.01 * N.shape[1]))
    for _ in range(case["iters"]):
        w, g = field(N)
        new = torch.where(g.norm(dim=0) > 0, -_unit(g), N)
        chord = (new - N).norm(dim=0)
        ang = torch.rad2deg(2 * torch.asin((0.5 * chord).clamp(max=1.0)))
        stats.append([float(w.mean()), float(torch.topk(ang, top).values.mean()), float(chord.mean())])
        N = new
    return {"N": N, "status": None, "stats": stats}


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        s = _train_state(case["rows"], seed)
        prm = s["params"].double().requires_grad_()
        y = _mlp64(prm, s["X"].double())
        cos = (y * s["T"].double()).sum(1) / y.norm(dim=1)
        keep = s["mask"] != 0
        loss = (1 - cos)[keep].sum() / max(1, int(keep.sum()))
        (g,) = torch.autograd.grad(loss, prm)
        m, v = 0.9 * s["m"].double() + 0.1 * g, 0.999 * s["v"].double() + 0.001 * g * g
        b1, b2 = 1 - 0.9 ** case["step"], 1 - 0.999 ** case["step"]
        new = prm.detach() - 1e-3 * (m / b1) / ((v / b2).sqrt() + 1e-8)
        return {"params": new, "m": m, "v": v, "loss": loss.detach().reshape(1), "grad": g}
    n = case["n"]
    if kind == "update":
        return None  # a level set's faces and their nearest points follow the field's signs
    if kind in ("areas", "knn") and n * (case.get("m") or n) > 2.5e10:
        return None  # all distances
    if kind in ("iterate", "field"):
        m, its = (case.get("m") or n), case.get("iters", 1)
        if (n * m * its > 1.5e10) if case["beta"] == 0.0 else (m * its * _interactions(n, case["beta"]) > 1e9):
            return None
    P, area, nv = _cloud(case["shape"], n, seed)
    if kind == "radius":
        return {"delta": _radius(P, case["k"])}
    if kind == "learned":
        return {"N": _unit(_mlp64(mlp_init.load_params(WEIGHTS, DEV).double(), _features(P)).T)}
    if kind == "areas":
        side = float((P.amax(1) - P.amin(1)).max())
        lo, hi = float(np.float32(0.0015 * side)), float(np.float32(0.015 * side))
        dist, idx = _near(P, P, 15, torch.arange(n, device=DEV))
        dist = dist[:, :10]
        ok = (dist >= lo) & (dist <= hi)
        mean = torch.where(ok, dist, 0.0).sum(1) / ok.sum(1).clamp_min(1)
        return {"area": _voronoi64(P, idx), "delta": torch.where(ok.any(1), mean, dist.mean(1).clamp(lo, hi))}
    if kind == "knn":
        Q = _queries(P, case["m"], seed) if case["m"] else P
        own = None if case["m"] else torch.arange(n, device=DEV)
        return {"idx": None, "dist": _near(Q, P, case["k"], own)[0]}
    dl, N = _radius(P).float(), _normals(nv, seed)
    Q = P if kind == "iterate" or not case["m"] else _queries(P, case["m"], seed)
    if case["beta"] == 0.0:
        field = lambda nrm: _all_pairs(P, nrm, area, dl, Q, case["lam"])  # noqa: E731
    else:
        tree = _Octree(P, area, dl, float(np.float32(case["beta"])))
        field = lambda nrm: tree.field(nrm, Q, case["lam"])  # noqa: E731
    if kind == "iterate":
        return _iterate64({"N": N}, case, field)
    w, g = field(N)
    return {"w": w, "grad": g} if case["grad"] else {"w": w}
