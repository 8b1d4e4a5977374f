"""FP64 points: chunks with and without edges that lead nowhere (loops of 3 to 29 edges over whole
and half chunks).  Four waves sharing 64 points, a lane per point and plans give the same bits; a
workgroup per point has the same terms in another order, 1e-16 each of at most some thousand; and
the direct sum over the triangles."""
import numpy as np
import pytest

import oracle as O
from paper_2605_01536_amd import workloads as W
from tests._util import fan_soup, off_surface_mask

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


SOUPS = {
    "fans": lambda: fan_soup([3, 4, 5, 6, 7, 8, 9, 10, 11, 13, 14, 15, 29, 3, 3, 5], 4),
    "triangle": lambda: (W.icosphere(2).V, W.icosphere(2).F[:1].copy()),
    "torus": lambda: (lambda s: (s.V, s.F))(W.torus_soup(seed=5, n_u=80, n_v=70)),   # over 4,096 edges
}


@pytest.mark.parametrize("soup", list(SOUPS))
def test_forms_agree_and_are_the_direct_sum(gwn, monkeypatch, soup):
    V, F = SOUPS[soup]()
    m = gwn.Mesh(_dev(V), _dev(F))
    rng = np.random.default_rng(3)
    lo, hi = V.min(0) - 0.1, V.max(0) + 0.1
    P = rng.uniform(lo, hi, (32769, 3)).astype(np.float32)
    P[::7, 2] = np.float32(hi[2] + 3)
    P[3::11] *= 50                                    # outside the box
    Q = _dev(P)
    w = gwn.query_batch(m, Q, prec="fp64")            # shared waves (the triangle: a lane per point)
    many = gwn.query_batch(m, Q.repeat(13, 1), prec="fp64")   # 425,997 points: a lane per point
    assert torch.equal(many.reshape(13, -1), w.expand(13, -1))
    for n in (1, 63, 64, 65, 8193):
        part = gwn.query_batch(m, Q[:n], prec="fp64")
        assert float((part - w[:n]).abs().max()) <= 1e-12
        assert torch.equal(part, w[:n]) or (soup == "torus" and n <= 8192)   # a workgroup per point
    monkeypatch.setenv("GWN_SPLIT_BOUNDARY", "1")
    assert float((gwn.query_batch(m, Q, prec="fp64") - w).abs().max()) <= 1e-12
    plan = gwn.MultiPlan([m, m], torch.cat([Q, Q[:777]]), [0, len(P), len(P) + 777], prec="fp64")
    plan.run()
    torch.cuda.synchronize()
    assert torch.equal(plan.w, torch.cat([w, w[:777]]))   # the lanes' sums, in their order
    pick = rng.choice(len(P), 400, replace=False)
    ok = off_surface_mask(V, F, P[pick])
    ref = O.direct(V, F, P[pick])
    assert np.abs(w.cpu().numpy()[pick] - ref)[ok].max() <= 1e-5   # the FP64 bar
