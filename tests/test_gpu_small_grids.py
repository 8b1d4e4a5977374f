"""Grids of few samples or little boundary around the lines between their forms: crossings from
lists or a walk per column, a column per wave or shared by eight, one to four samples per lane.
Counts are a query's; w is a query's up to the order of at most a few hundred terms (FP64:
1e-16 each, FP32: a tenth of its bar)."""
import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _one():
    s = W.icosphere(2)
    s.F = s.F[:1].copy()
    return s


SOUPS = {
    "triangle": _one,                                                      # 1 chunk: never lists, never shared
    "closed320": lambda: W.icosphere(2),                                   # lists from some 9,600 waves on
    "closed5k": lambda: W.icosphere(4),
    "spheres": lambda: W.opened_spheres(seed=1, n_surf=4, tris_per_surf=400),        # about 10 chunks
    "spheres8": lambda: W.opened_spheres(seed=1, n_surf=8, tris_per_surf=400),       # about 20
    "ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(1), 1000, 0.1),    # about 36
}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("soup", list(SOUPS))
@pytest.mark.parametrize("dims", [(3, 5, 7), (16, 15, 9), (25, 24, 130), (40, 37, 3), (66, 65, 2), (100, 97, 2), (7, 9, 190)])
def test_counts_and_sums_are_the_points(gwn, soup, dims, prec):
    s = SOUPS[soup]()
    m = gwn.Mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda())
    lo, hi = s.bbox()
    lo, hi = lo - 0.07, hi + 0.06
    for flip in (1, -1):   # falling z: no lists
        sp = (hi - lo) / np.array(dims) * np.array([1, 1, flip])
        o = np.array([lo[0], lo[1], lo[2] if flip > 0 else hi[2]])
        g = tuple(float(x) for x in o), tuple(float(x) for x in sp), dims
        w, c = gwn.query_grid(m, *g, prec=prec, want_chi=True)
        P = torch.from_numpy(W.grid_points(W.GridSpec(*g))).cuda()
        wb, cb = gwn.query_batch(m, P, prec=prec, want_chi=True)
        assert torch.equal(c.reshape(-1), cb)
        assert float((w.reshape(-1).double() - wb.double()).abs().max()) <= (1e-5 if prec == "fp32" else 1e-11)
