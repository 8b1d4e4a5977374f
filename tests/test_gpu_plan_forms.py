"""Multi-mesh plans whatever the form of their kernels (crossings by ordered waves, a lane or a wave
per query; sums by ordered or unordered lanes, in groups): the same bits as the single-mesh calls,
also where launches are cut into slices of few items and where the queries are not those that the
orders were made from."""
import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _mesh(gwn, s):
    return gwn.Mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda())


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_sliced_launches(gwn, monkeypatch, prec):
    soups = [W.torus_soup(seed=3, n_u=40, n_v=30), W.ellipsoid_union(np.random.default_rng(4), 900, 0.1),
             W.icosphere(2), W.opened_spheres(seed=2, n_surf=3, tris_per_surf=400)]
    sizes = [17001, 4000, 1, 300]   # in order, and not
    rng = np.random.default_rng(5)
    Q = torch.from_numpy(np.concatenate([W.uniform_box(rng, n, *s.bbox()) for n, s in zip(sizes, soups)])).cuda()
    off = np.concatenate([[0], np.cumsum(sizes)])
    meshes = [_mesh(gwn, s) for s in soups]
    ref = gwn.MultiPlan(meshes, Q, off, prec=prec)
    ref.run()
    monkeypatch.setenv("GWN_MAX_LAUNCH_QUERIES", "256")   # one item per launch
    chi = torch.full((len(Q),), -99, dtype=torch.int32, device="cuda")
    plan = gwn.MultiPlan(meshes, Q, off, chi_out=chi, prec=prec)
    for _ in range(2):
        plan.w.fill_(-7)
        chi.fill_(-99)
        plan.run()
        torch.cuda.synchronize()
        assert torch.equal(plan.w, ref.w)
    monkeypatch.delenv("GWN_MAX_LAUNCH_QUERIES")
    for i, m in enumerate(meshes):
        _, c = gwn.query_batch(m, Q[off[i]:off[i + 1]], want_chi=True)
        assert torch.equal(chi[off[i]:off[i + 1]], c)


def _strip(n):
    """two rows of n + 1 vertices: one loop of 2 n + 2 edges"""
    x = np.linspace(0, 1, n + 1)
    c = np.stack([np.cos(9 * x) * (1 + x), np.sin(9 * x) * (1 + x), x], 1)
    i = np.arange(n)
    F = np.concatenate([np.stack([i, i + 1, n + 1 + i], 1), np.stack([i + 1, n + 2 + i, n + 1 + i], 1)])
    return W.Soup(V=np.concatenate([c, c * [0.9, 0.9, 1] + [0, 0, 0.05]]).astype(np.float32), F=F.astype(np.int32))


def _triangle():
    s = W.icosphere(2)
    s.F = s.F[:1].copy()
    return s


SOUPS = {
    "triangle": _triangle,
    "closed": lambda: W.icosphere(3),
    "spheres": lambda: W.opened_spheres(seed=1, n_surf=4, tris_per_surf=400),          # few wide edges
    "strip": lambda: _strip(700),                                                      # one cluster, a long loop
    "ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(2), 4000, 0.1),      # some 1,000 edges
    "torus": lambda: W.torus_soup(seed=2, n_u=130, n_v=100),                           # some 16,000
}


# few queries in all (a wave each, groups); many of meshes that are short of an order (lanes); both
# sides of an order's 16,384
@pytest.mark.parametrize("sizes", [(1, 63, 64, 65, 700, 129), (4000, 9000, 16383, 8193, 12000, 5000),
                                   (16384, 16384, 16385, 16384, 16384, 16384)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("order", [0, 2])
def test_forms(gwn, monkeypatch, sizes, prec, order):
    monkeypatch.setenv("GWN_SPLIT_BOUNDARY", "0")   # FP64: a lane per point
    soups = [f() for f in SOUPS.values()]
    meshes = [_mesh(gwn, s) for s in soups]
    rng = np.random.default_rng(6)
    Q = [torch.from_numpy(W.uniform_box(rng, n, s.bbox()[0] - 0.1, s.bbox()[1] + 0.1)).cuda() for n, s in zip(sizes, soups)]
    ref = [gwn.query_batch(m, q, prec=prec, want_chi=True) for m, q in zip(meshes, Q)]
    w, c = (torch.cat([r[k] for r in ref]) for k in (0, 1))
    Q = torch.cat(Q)
    chi = torch.full((len(Q),), -99, dtype=torch.int32, device="cuda")
    late = torch.zeros_like(Q)
    off = np.concatenate([[0], np.cumsum(sizes)])
    for q in (Q, late):
        plan = gwn.MultiPlan(meshes, q, off, chi_out=chi, order=order, prec=prec)
        late.copy_(Q)
        for _ in range(2):
            plan.w.fill_(-7)
            chi.fill_(-99)
            torch.cuda.synchronize()
            plan.run()
            torch.cuda.synchronize()
            assert torch.equal(plan.w, w) and torch.equal(chi, c)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_many_unordered_queries(gwn, prec):
    """enough of them that small and closed meshes' crossings are a lane's; the others' a wave's"""
    pool = [(_mesh(gwn, s), s) for s in (SOUPS[k]() for k in ("closed", "spheres", "ellipsoids"))]
    rng = np.random.default_rng(7)
    sizes = [16383] * 17 + [1]
    meshes, Q, w, c = [], [], [], []
    for i, n in enumerate(sizes):
        m, s = pool[i % 3]
        q = torch.from_numpy(W.uniform_box(rng, n, s.bbox()[0] - 0.1, s.bbox()[1] + 0.1)).cuda()
        a, b = gwn.query_batch(m, q, prec=prec, want_chi=True)
        meshes.append(m), Q.append(q), w.append(a), c.append(b)
    Q = torch.cat(Q)
    chi = torch.full((len(Q),), -99, dtype=torch.int32, device="cuda")
    plan = gwn.MultiPlan(meshes, Q, np.concatenate([[0], np.cumsum(sizes)]), chi_out=chi, prec=prec)
    plan.run()
    torch.cuda.synchronize()
    assert torch.equal(plan.w, torch.cat(w)) and torch.equal(chi, torch.cat(c))
