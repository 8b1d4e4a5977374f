"""Grids in boxes of samples, launched in slices: the same bits as in one launch."""
import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(5, 7, 8), (20, 20, 20), (37, 20, 29)])   # 16, 16 and 8 waves a box
def test_sliced_boxes(gwn, monkeypatch, dims):
    s = W.ellipsoid_union(np.random.default_rng(5), 4000, 0.1)
    m = gwn.Mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda())
    monkeypatch.setenv("GWN_GRID_BOXES", "1")
    lo, hi = s.bbox()
    g = tuple(float(x) for x in lo), tuple(float(x) for x in (hi - lo) / np.array(dims)), dims
    w0, c0 = gwn.query_grid(m, *g, want_chi=True)
    P = torch.from_numpy(W.grid_points(W.GridSpec(*g))).cuda()
    assert torch.equal(w0.reshape(-1), gwn.query_batch(m, P))   # in boxes: the points' bits
    for most in ("256", "2048"):
        monkeypatch.setenv("GWN_MAX_LAUNCH_QUERIES", most)
        w1 = torch.full_like(w0, -7)
        w1, c1 = gwn.query_grid(m, *g, want_chi=True, out=w1)
        assert torch.equal(w0, w1) and torch.equal(c0, c1)
