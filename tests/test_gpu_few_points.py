"""FP32 batches of few points, a workgroup for each (up to 256): the bits of a lane per point, on
soups of far clusters of every degree, near ones, and a loop of thousands of chunks; points above,
below and outside the fixed-point box, at heights beyond shared arctangents."""
import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _strip(n):
    x = np.linspace(0, 1, n + 1)
    c = np.stack([np.cos(9 * x) * (1 + x), np.sin(9 * x) * (1 + x), x], 1)
    i = np.arange(n)
    F = np.concatenate([np.stack([i, i + 1, n + 1 + i], 1), np.stack([i + 1, n + 2 + i, n + 1 + i], 1)])
    return W.Soup(V=np.concatenate([c, c * [0.9, 0.9, 1] + [0, 0, 0.05]]).astype(np.float32), F=F.astype(np.int32))


def _both():
    a, b = _strip(15000), W.torus_soup(seed=2, n_u=60, n_v=50)
    return W.Soup(V=np.concatenate([a.V, b.V]), F=np.concatenate([a.F, b.F + len(a.V)]))


SOUPS = {"loop": lambda: _strip(20000), "torus": lambda: W.torus_soup(seed=2, n_u=130, n_v=100), "loop and torus": _both,
         "ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(2), 4000, 0.1)}


@pytest.mark.parametrize("soup", list(SOUPS))
def test_bits_of_a_lane_per_point(gwn, monkeypatch, soup):
    s = SOUPS[soup]()
    m = gwn.Mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda())
    rng = np.random.default_rng(1)
    lo, hi = s.bbox()
    P = rng.uniform(lo - 0.05, hi + 0.05, (600, 3)).astype(np.float32)
    P[::9, 2] = hi[2] + rng.uniform(0, 4, len(P[::9]))
    P[1::9, 2] = lo[2] - rng.uniform(0, 4, len(P[1::9]))
    P[2::37] *= 60
    P[3::41, 2] = 300 * rng.choice([-1, 1], len(P[3::41]))
    Q = torch.from_numpy(P).cuda()
    monkeypatch.setenv("GWN_SPLIT_BOUNDARY", "0")
    w = gwn.query_batch(m, Q)
    monkeypatch.delenv("GWN_SPLIT_BOUNDARY")
    for n in (1, 2, 255, 256, 257, 600):
        assert torch.equal(gwn.query_batch(m, Q[:n]), w[:n]), n


# few, wide edges: up to 16,384 points 16 waves share 64, then four, above 2^20 none
@pytest.mark.parametrize("soup", ["spheres", "ellipsoids", "more ellipsoids"])
def test_bits_of_shared_lanes_on_few_edges(gwn, soup):
    s = {"spheres": lambda: W.opened_spheres(seed=1, n_surf=4, tris_per_surf=400),
         "ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(1), 1000, 0.1),
         "more ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(4), 1300, 0.1)}[soup]()
    m = gwn.Mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda())
    rng = np.random.default_rng(3)
    lo, hi = s.bbox()
    P = rng.uniform(lo - 0.05, hi + 0.05, (2 ** 20 + 1, 3)).astype(np.float32)
    P[2::37] *= 60
    P[3::41, 2] = 300 * rng.choice([-1, 1], len(P[3::41]))
    Q = torch.from_numpy(P).cuda()
    w = gwn.query_batch(m, Q)
    for n in (1, 63, 64, 65, 1063, 16384, 16385):
        assert torch.equal(gwn.query_batch(m, Q[:n]), w[:n]), n
        if n <= 1063:
            assert torch.equal(gwn.query_batch_noalloc(m, Q[:n]), w[:n]), n
