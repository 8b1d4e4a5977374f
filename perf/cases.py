"""The timed work of this framework: generalized winding numbers of triangle soups on grids and at
points, their gradient, plans over many soups, the preparation of a soup, the learned surrogate and
Bezier surfaces, each through the public calls of ``paper_2605_01536_amd.gwn``.

A case is a dict of plain values; ``kind`` names the call, the rest its sizes:

* ``grid``            query_grid on a cell-centred grid, FP32 or FP64
* ``grid_gradient``   query_grid_gradient
* ``points``          query_batch at scattered points, FP32 or FP64, crossing counts on request
* ``plan``            MultiPlan.run over many soups of uneven size (one captured graph)
* ``build``           a soup as a file stores it (three vertices of its own per triangle): Mesh with
                      welding and the automatic ray axis, then a first small batch
* ``infer``           Surrogate.forward
* ``loss_grad``       Surrogate.loss_grad: one mini-batch forward and backward
* ``bezier``          Patches.query_grid

Soups: ``spheres`` (overlapping opened spheres and ellipsoids, one smooth boundary loop each),
``torus`` (a noisy torus with a fifth of its triangles missing: a ragged boundary all over),
``ellipsoids`` (a union of ellipsoids with a tenth of the triangles missing) and ``closed`` (an
icosphere without a boundary).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_01536_amd import gwn
from paper_2605_01536_amd import workloads as wl


def listed():
    return [
        # a dense voxelisation of a large open soup: the workload that the throughput is quoted on
        {"name": "grid_512_fp32", "kind": "grid", "prec": "fp32", "soup": "spheres", "tris": 19600, "surfs": 64,
         "nx": 512, "ny": 512, "nz": 512},
        # an interactive preview of a small model: launches and latency count
        {"name": "grid_small_fp32", "kind": "grid", "prec": "fp32", "soup": "ellipsoids", "tris": 4000, "surfs": 0,
         "nx": 37, "ny": 50, "nz": 29},
        # a double-precision field of a medium model on a box of unequal sides
        {"name": "grid_medium_fp64", "kind": "grid", "prec": "fp64", "soup": "ellipsoids", "tris": 30000, "surfs": 0,
         "nx": 120, "ny": 97, "nz": 121},
        # the field's gradient on a volume, as reconstruction and meshing codes sample it
        {"name": "grid_gradient_fp32", "kind": "grid_gradient", "prec": "fp32", "soup": "spheres", "tris": 4900,
         "surfs": 32, "nx": 192, "ny": 200, "nz": 177},
        # a handful of containment tests against a small closed model: the smallest call
        {"name": "points_few_closed", "kind": "points", "prec": "fp32", "soup": "closed", "tris": 1280, "surfs": 0,
         "points": 1000, "near": False, "chi": False},
        # a few thousand samples of a ragged scan, with the crossing counts
        {"name": "points_4k_fp32_chi", "kind": "points", "prec": "fp32", "soup": "torus", "tris": 100000, "surfs": 0,
         "points": 4099, "near": False, "chi": True},
        # a point cloud, half of it near the surface, against the same kind of scan
        {"name": "points_2m_fp32", "kind": "points", "prec": "fp32", "soup": "torus", "tris": 100000, "surfs": 0,
         "points": 2000000, "near": True, "chi": False},
        # a data set of soups evaluated again and again by one captured plan
        {"name": "plan_48_soups", "kind": "plan", "meshes": 48, "tris": 50000, "points": 200000},
        # a model arrives as a triangle file: weld, prepare, first answers
        {"name": "build_weld_first_batch", "kind": "build", "soup": "spheres", "tris": 9216, "surfs": 40,
         "points": 2000},
        # the learned surrogate over a large point set
        {"name": "infer_16m", "kind": "infer", "points": 16000000},
        # one mini-batch of the surrogate's training, forward and backward
        {"name": "loss_grad_8192", "kind": "loss_grad", "points": 8192},
        # a CAD surface of free-form patches voxelised in double precision
        {"name": "bezier_100_grid_32", "kind": "bezier", "patches": 100, "nx": 32, "ny": 32, "nz": 32},
    ]


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["grid", "grid", "grid", "grid_gradient", "points", "points", "points", "plan", "build",
                       "infer", "loss_grad", "bezier"])
    if kind in ("grid", "grid_gradient"):
        soup = rng.choice(["spheres", "ellipsoids", "torus"])
        tris, surfs = {"spheres": (log(400, 19600), rng.randint(4, 64)), "ellipsoids": (log(1000, 200000), 0),
                       "torus": (log(2000, 100000), 0)}[soup]
        # soups with a ragged boundary get smaller grids: the cost goes with samples x boundary edges
        hi = {"spheres": 384, "ellipsoids": 200, "torus": 160}[soup] if kind == "grid" else 160
        return {"kind": kind, "prec": rng.choice(["fp32", "fp32", "fp64"]), "soup": soup, "tris": tris,
                "surfs": surfs, "nx": log(20, hi), "ny": log(20, hi), "nz": log(20, hi)}
    if kind == "points":
        soup = rng.choice(["spheres", "ellipsoids", "torus", "closed"])
        tris, surfs = {"spheres": (log(400, 19600), rng.randint(4, 64)), "ellipsoids": (log(1000, 200000), 0),
                       "torus": (log(2000, 100000), 0), "closed": (rng.choice([320, 1280, 5120]), 0)}[soup]
        return {"kind": kind, "prec": rng.choice(["fp32", "fp32", "fp64"]), "soup": soup, "tris": tris,
                "surfs": surfs, "points": log(500, 2000000), "near": rng.random() < 0.5,
                "chi": rng.random() < 0.3}
    if kind == "plan":
        return {"kind": kind, "meshes": rng.randint(8, 48), "tris": log(5000, 50000), "points": log(20000, 200000)}
    if kind == "build":
        soup = rng.choice(["spheres", "torus", "ellipsoids"])
        tris, surfs = {"spheres": (log(400, 9216), rng.randint(8, 40)), "ellipsoids": (log(5000, 300000), 0),
                       "torus": (log(5000, 200000), 0)}[soup]
        return {"kind": kind, "soup": soup, "tris": tris, "surfs": surfs, "points": log(500, 4000)}
    if kind == "infer":
        return {"kind": kind, "points": log(10000, 16000000)}
    if kind == "loss_grad":
        return {"kind": kind, "points": log(2000, 131072)}
    return {"kind": "bezier", "patches": log(8, 100), "nx": log(8, 32), "ny": log(8, 32), "nz": log(8, 32)}


# ---------------------------------------------------------------- inputs, from the seed alone

def _soup(case, seed):
    kind, tris = case["soup"], case["tris"]
    if kind == "closed":
        s = wl.icosphere({320: 2, 1280: 3, 5120: 4}[tris])
        rng = np.random.default_rng(seed)   # another size and place for each seed
        s.V = (s.V * rng.uniform(0.5, 1.5) + rng.uniform(-0.2, 0.2, 3)).astype(np.float32)
        return s
    if kind == "spheres":
        return wl.opened_spheres(seed=seed, n_surf=case["surfs"], tris_per_surf=tris)
    if kind == "torus":
        n_v = max(8, int(round(math.sqrt(tris / 2 / 1.25))))
        return wl.torus_soup(seed=seed, n_u=max(10, int(round(tris / 2 / n_v))), n_v=n_v)
    return wl.ellipsoid_union(np.random.default_rng(seed), tris, 0.1)


def _points(case, soup, seed):
    rng = np.random.default_rng([seed, 1])
    n = case["points"]
    lo, hi = soup.bbox()
    if case["soup"] == "closed":
        lo, hi = lo - 0.5, hi + 0.5
    if not case.get("near"):
        return wl.uniform_box(rng, n, lo, hi)
    sigma = 1e-3 * float(np.linalg.norm(hi - lo))
    Q = np.concatenate([wl.uniform_box(rng, n - n // 2, lo, hi), wl.near_surface(rng, soup, n // 2, sigma)])
    return Q


def _grid(case, soup):
    """The cell-centred grid over the soup's box with a margin of 5%."""
    lo, hi = soup.bbox()
    pad = 0.05 * (hi - lo).max()
    dims = (case["nx"], case["ny"], case["nz"])
    lo, hi = lo - pad, hi + pad
    return tuple(float(x) for x in lo), tuple(float((hi[a] - lo[a]) / dims[a]) for a in range(3)), dims


def _plan(case, seed):
    """The sizes of the soups and of their point sets belong to the case, the shapes to the seed."""
    sizes, rng = np.random.default_rng(case["meshes"]), np.random.default_rng(seed)
    soups, queries = [], []
    for _ in range(case["meshes"]):
        nt = int(round(math.exp(sizes.uniform(math.log(1000), math.log(case["tris"])))))
        nq = int(round(math.exp(sizes.uniform(math.log(10000), math.log(case["points"])))))
        s = wl.ellipsoid_union(rng, nt, rng.uniform(0.0, 0.3))
        soups.append(s)
        queries.append(wl.uniform_box(rng, nq, *s.bbox()))
    return soups, queries


def _patches(case, seed):
    return np.random.default_rng(seed).uniform(0.0, 1.0, size=(case["patches"], 16, 3))


def _box_points(n, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 40))
    return torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float32) * 2.0 - 1.0


def _labels(Q):
    """Inside or outside a ball: labels of the kind that the surrogate learns."""
    return (Q.square().sum(1) < 0.5).to(torch.float32)


def _mesh(soup, **kw):
    return gwn.build_mesh(torch.from_numpy(soup.V).cuda(), torch.from_numpy(soup.F).cuda(), **kw)


def prepare(case, seed):
    kind, st = case["kind"], {"case": case}
    if kind in ("grid", "grid_gradient"):
        s = _soup(case, seed)
        st["mesh"] = _mesh(s)
        st["grid"] = _grid(case, s)
    elif kind == "points":
        s = _soup(case, seed)
        st["mesh"] = _mesh(s)
        st["Q"] = torch.from_numpy(_points(case, s, seed)).cuda()
    elif kind == "plan":
        soups, queries = _plan(case, seed)
        st["meshes"] = [_mesh(s) for s in soups]
        off = np.concatenate([[0], np.cumsum([len(q) for q in queries])])
        st["plan"] = gwn.MultiPlan(st["meshes"], torch.from_numpy(np.concatenate(queries)).cuda(), off.tolist())
    elif kind == "build":
        s = _soup(case, seed)
        e = wl.explode(s, seed=int(seed) % (1 << 31))
        st["V"], st["F"] = torch.from_numpy(e.V).cuda(), torch.from_numpy(e.F).cuda()
        st["Q"] = torch.from_numpy(_points(case, s, seed)).cuda()
    elif kind == "bezier":
        st["P"] = gwn.Patches(torch.from_numpy(_patches(case, seed)).cuda())
        st["grid"] = ((-0.2,) * 3, tuple(1.4 / case[a] for a in ("nx", "ny", "nz")),
                      (case["nx"], case["ny"], case["nz"]))
    else:
        st["net"] = gwn.Surrogate(seed=int(seed) % (1 << 31), sigma=1.0)
        st["Q"] = _box_points(case["points"], seed)
        if kind == "loss_grad":
            st["T"] = _labels(st["Q"])
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "grid":
        return gwn.query_grid(st["mesh"], *st["grid"], prec=case["prec"])
    if kind == "grid_gradient":
        return gwn.query_grid_gradient(st["mesh"], *st["grid"], prec=case["prec"])
    if kind == "points":
        return gwn.query_batch(st["mesh"], st["Q"], prec=case["prec"], want_chi=case["chi"])
    if kind == "plan":
        return st["plan"].run()
    if kind == "build":
        m = gwn.build_mesh(st["V"], st["F"], weld=True, axis="auto")
        w = gwn.query_batch(m, st["Q"])
        i = m.info()
        m.close()
        return w, i["nboundary"], i["nloops"], i["nunique"]
    if kind == "infer":
        return st["net"].forward(st["Q"])
    if kind == "loss_grad":
        return st["net"].loss_grad(st["Q"], st["T"])
    return st["P"].query_grid(*st["grid"])


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Every input and output once; as operations a constant number per output value and per triangle
    (the sum over the boundary is no lower bound: parts of it that are far away can be shared), for the
    network its matrix products, for patches 100 of each of a sample's curves."""
    kind = case["kind"]
    if kind in ("infer", "loss_grad"):
        n, f = case["points"], 2 * (64 * 128 + 3 * 128 * 128 + 128 + 32 * 3)
        if kind == "infer":
            return {"bytes": 16 * n, "flops": f * n}
        return {"bytes": 16 * n + 8 * 57985, "flops": 3 * f * n}
    if kind == "bezier":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 8 * n + 384 * case["patches"], "flops": 100 * 4 * case["patches"] * n}
    if kind == "plan":   # expected sizes of the log-uniform draws
        def mean(lo, hi):
            return (hi - lo) / math.log(hi / lo) if hi > lo else lo
        nq, nt = case["meshes"] * mean(10000, case["points"]), case["meshes"] * mean(1000, case["tris"])
        return {"bytes": int(16 * nq + 18 * nt), "flops": int(100 * nq + 100 * nt)}
    nt = case["tris"] * max(1, case["surfs"])
    if kind == "build":
        return {"bytes": 48 * nt + 16 * case["points"], "flops": 100 * nt}
    size = 8 if case["prec"] == "fp64" else 4
    if kind == "points":
        n = case["points"]
        return {"bytes": (12 + size + 4 * bool(case["chi"])) * n + 18 * nt, "flops": 100 * n + 100 * nt}
    n = case["nx"] * case["ny"] * case["nz"]
    return {"bytes": size * (3 if kind == "grid_gradient" else 1) * n + 18 * nt, "flops": 100 * n + 100 * nt}


# ---------------------------------------------------------------- the same values in 64 bits

_PAIRS = 4e10      # (point, triangle) or (point, boundary edge) pairs that fit the time


def _solid_angles(V, F, Q):
    """Sum over the triangles of the signed solid angle over 4 pi (Van Oosterom and Strackee)."""
    T = torch.as_tensor(V[F], dtype=torch.float64, device="cuda")          # (nf, 3, 3)
    Q = torch.as_tensor(Q, dtype=torch.float64, device="cuda")
    out = torch.zeros(Q.shape[0], dtype=torch.float64, device="cuda")
    nt = min(T.shape[0], 4096)
    nq = max(1, (1 << 25) // nt)
    for q0 in range(0, Q.shape[0], nq):
        q = Q[q0:q0 + nq, None, :]
        for t0 in range(0, T.shape[0], nt):
            t = T[t0:t0 + nt]
            a, b, c = ([t[None, :, k, d] - q[:, :, d] for d in range(3)] for k in range(3))
            la, lb, lc = (torch.sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]) for x in (a, b, c))
            num = (a[0] * (b[1] * c[2] - b[2] * c[1]) + a[1] * (b[2] * c[0] - b[0] * c[2])
                   + a[2] * (b[0] * c[1] - b[1] * c[0]))
            ab, bc, ca = (x[0] * y[0] + x[1] * y[1] + x[2] * y[2] for x, y in ((a, b), (b, c), (c, a)))
            out[q0:q0 + nq] += torch.atan2(num, la * lb * lc + ab * lc + bc * la + ca * lb).sum(1)
    return out / (2.0 * math.pi)


def _field(V, F, Q):
    """The gradient: the Biot-Savart field of the boundary's segments over 4 pi."""
    E = np.concatenate([F[:, [0, 1]], F[:, [1, 2]], F[:, [2, 0]]]).astype(np.int64)
    lo, hi = E.min(1), E.max(1)
    key, inv = np.unique(lo * V.shape[0] + hi, return_inverse=True)
    net = np.bincount(inv.ravel(), weights=np.where(E[:, 0] == lo, 1.0, -1.0), minlength=len(key))
    keep = net != 0
    A = torch.as_tensor(V[key[keep] // V.shape[0]], dtype=torch.float64, device="cuda")
    B = torch.as_tensor(V[key[keep] % V.shape[0]], dtype=torch.float64, device="cuda")
    m = torch.as_tensor(net[keep], dtype=torch.float64, device="cuda")
    if Q.shape[0] * A.shape[0] > _PAIRS:
        return None
    Q = torch.as_tensor(Q, dtype=torch.float64, device="cuda")
    out = torch.zeros((Q.shape[0], 3), dtype=torch.float64, device="cuda")
    ne = min(max(1, A.shape[0]), 4096)
    nq = max(1, (1 << 25) // ne)
    for q0 in range(0, Q.shape[0], nq):
        q = Q[q0:q0 + nq, None, :]
        for e0 in range(0, A.shape[0], ne):
            a = [A[None, e0:e0 + ne, d] - q[:, :, d] for d in range(3)]
            b = [B[None, e0:e0 + ne, d] - q[:, :, d] for d in range(3)]
            la = torch.sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2])
            lb = torch.sqrt(b[0] * b[0] + b[1] * b[1] + b[2] * b[2])
            f = (la + lb) / (la * lb * (la * lb + a[0] * b[0] + a[1] * b[1] + a[2] * b[2])) * m[None, e0:e0 + ne]
            for d in range(3):
                i, j = (d + 1) % 3, (d + 2) % 3
                out[q0:q0 + nq, d] += ((a[i] * b[j] - a[j] * b[i]) * f).sum(1)
    return out / (4.0 * math.pi)


def _network(st, Q):
    """The network's parameters (leaves) and its outputs at Q, in 64 bits with the exact GELU."""
    s = st["net"].state()
    th = torch.as_tensor(s["theta"], dtype=torch.float64, device="cuda").requires_grad_(True)
    z = 2.0 * math.pi * (Q.double() @ torch.as_tensor(s["G"], dtype=torch.float64, device="cuda").T)
    x, o = torch.cat([torch.sin(z), torch.cos(z)], 1), 0
    for i, (a, b) in enumerate(((64, 128), (128, 128), (128, 128), (128, 128), (128, 1))):
        x = x @ th[o:o + a * b].view(a, b) + th[o + a * b:o + a * b + b]
        o += a * b + b
        if i < 4:
            x = torch.nn.functional.gelu(x)
    return th, x[:, 0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "bezier":
        return None   # an adaptive quadrature to 1e-12 at every sample takes minutes
    if kind == "infer":
        st = prepare(case, seed)
        with torch.no_grad():
            return torch.cat([_network(st, q)[1] for q in st["Q"].split(1 << 20)])
    if kind == "loss_grad":
        st = prepare(case, seed)
        th, y = _network(st, st["Q"])
        loss = (y - st["T"].double()).square().mean()
        return float(loss), torch.autograd.grad(loss, th)[0]
    if kind == "plan":
        soups, queries = _plan(case, seed)
        if sum(s.nf * len(q) for s, q in zip(soups, queries)) > _PAIRS:
            return None
        return torch.cat([_solid_angles(s.V, s.F, q) for s, q in zip(soups, queries)])
    s = _soup(case, seed)
    if kind in ("grid", "grid_gradient"):
        g = wl.GridSpec(*_grid(case, s))
        n = g.n
        if kind == "grid":
            return _solid_angles(s.V, s.F, wl.grid_points(g)) if n * s.nf <= _PAIRS else None
        return _field(s.V, s.F, wl.grid_points(g))
    Q = _points(case, s, seed)
    if len(Q) * s.nf > _PAIRS:
        return None
    w = _solid_angles(s.V, s.F, Q)
    if kind == "build":
        return w, None, None, None
    return (w, None) if case["chi"] else w
