"""FP32 sums have the same bits in every form also for points outside the fixed-point box in x or y
and far below it, where the edges' terms do not fall with the distance, on meshes near the origin
and far from it (where coordinates are large and distances small)."""
import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("soup", ["torus", "spheres", "ellipsoids"])
@pytest.mark.parametrize("shift", [0.0, 3000.0])
def test_bits_beside_and_far_below(gwn, monkeypatch, soup, shift):
    s = {"torus": lambda: W.torus_soup(seed=2, n_u=130, n_v=100),
         "spheres": lambda: W.opened_spheres(seed=2, n_surf=6, tris_per_surf=4000),
         "ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(2), 4000, 0.1)}[soup]()
    V = (s.V + np.float32(shift)).astype(np.float32)
    m = gwn.Mesh(torch.from_numpy(V).cuda(), torch.from_numpy(s.F).cuda())
    lo, hi = V.min(0).astype(np.float64), V.max(0).astype(np.float64)
    e = float((hi - lo).max())
    rng = np.random.default_rng(1)
    n = 7000
    P = rng.uniform(lo, hi, (n, 3))
    out = rng.integers(0, 2, n)
    P[np.arange(n), out] = np.where(rng.random(n) < 0.5, lo[out] - e * rng.uniform(0.76, 1.5, n), hi[out] + e * rng.uniform(0.76, 1.5, n))
    P[:, 2] = lo[2] - e * 10.0 ** rng.uniform(0, 11, n)
    P[::7, 2] = hi[2] + e * 10.0 ** rng.uniform(0, 11, len(P[::7]))      # above
    P[::11, 0] = lo[0] - e * 10.0 ** rng.uniform(0, 11, len(P[::11]))    # far beside
    Q = torch.from_numpy(P.astype(np.float32)).cuda()
    monkeypatch.setenv("GWN_SPLIT_BOUNDARY", "0")
    w = gwn.query_batch(m, Q)                                  # a lane per point
    monkeypatch.setenv("GWN_SPLIT_BOUNDARY", "1")
    assert torch.equal(gwn.query_batch(m, Q), w)               # groups, a wave, a workgroup per point
    assert torch.equal(gwn.query_batch(m, Q[:5000]), w[:5000])
    assert torch.equal(gwn.query_batch(m, Q[:200]), w[:200])
    monkeypatch.delenv("GWN_SPLIT_BOUNDARY")
    plan = gwn.MultiPlan([m, m], torch.cat([Q, Q, Q, Q]), [0, n, 4 * n])
    plan.run()
    torch.cuda.synchronize()
    assert torch.equal(plan.w.reshape(4, n), w.expand(4, n))
