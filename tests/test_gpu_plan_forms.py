"""Multi-mesh plans whatever the form of their kernels: the same bits as the single-mesh calls
where launches are cut into slices of few items."""
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
