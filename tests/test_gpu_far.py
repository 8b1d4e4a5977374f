"""The grid path's far part (chunk sums at nodes, interpolated) and its crossing
lists against the sum over all chunks with a BVH walk per column, and against the
oracle: block sizes forced where grids are small, ragged last blocks, axes with fewer
samples than nodes, every ray axis and falling coordinates, columns of more crossings
than a list holds, capture.  The two sums differ by the interpolation (at most 2e-7 of
the terms of the chunks nearest to far in FP32, 6e-13 in FP64) and by rounding in
another order; the bound is a tenth of the FP32 bar, and 1e-11 in FP64."""
import numpy as np
import pytest

import oracle as O

from paper_2605_01536_amd import workloads as W
from tests._util import TOL_FP32, TOL_FP64, compare, fan_soup

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SAME = {"fp32": 1e-5, "fp64": 1e-11}


def _mesh(gwn, V, F, **kw):
    return gwn.Mesh(torch.from_numpy(np.ascontiguousarray(V)).cuda(), torch.from_numpy(np.ascontiguousarray(F)).cuda(),
                    **kw)


def _grid(V, dims, flip=(1, 1, 1)):
    lo, hi = V.min(0).astype(np.float64) - 0.05, V.max(0).astype(np.float64) + 0.05
    sp = (hi - lo) / np.array(dims)
    o = np.where(np.array(flip) > 0, lo, hi)
    return tuple(o), tuple(sp * np.array(flip)), dims


SOUPS = {
    "spheres": lambda: W.opened_spheres(seed=9, n_surf=6, tris_per_surf=900),
    "torus": lambda: W.torus_soup(seed=5, n_u=40, n_v=30),
    "ellipsoids": lambda: W.ellipsoid_union(np.random.default_rng(3), 3000, 0.1),
    # loops of 2 (a fan of two), 3, 7, 8, 14 and 15 edges: rests and whole chunks
    "fans": lambda: W.Soup(*fan_soup([3, 7, 8, 14, 15, 4, 3, 6, 29, 64], 4)),
}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("soup,dims,block,axis,flip", [
    ("spheres", (40, 33, 65), 8, "z", (1, 1, 1)),
    ("spheres", (17, 41, 130), 10, "x", (1, 1, 1)),      # last blocks of one sample
    ("torus", (48, 48, 12), 12, "z", (1, 1, 1)),          # z: 12 samples, FP64 all of them nodes
    ("torus", (64, 1, 64), 8, "y", (1, 1, 1)),            # a slice: one sample in a column direction
    ("ellipsoids", (33, 9, 50), 8, "z", (-1, 1, -1)),     # falling coordinates (no crossing lists)
    ("ellipsoids", (70, 70, 20), 16, "x", (1, -1, 1)),
    ("fans", (31, 29, 257), 8, "z", (1, 1, 1)),
])
def test_far_part_equals_all_chunks(gwn, monkeypatch, prec, soup, dims, block, axis, flip):
    s = SOUPS[soup]()
    m = _mesh(gwn, s.V, s.F, axis=axis)
    g = _grid(s.V, dims, flip)
    monkeypatch.setenv("GWN_GRID_FAR", "0")
    w0, c0 = gwn.query_grid(m, *g, prec=prec, want_chi=True)
    monkeypatch.setenv("GWN_GRID_FAR", str(block))
    w1, c1 = gwn.query_grid(m, *g, prec=prec, want_chi=True)
    assert torch.equal(gwn.query_grid(m, *g, prec=prec), w1)
    assert torch.equal(c0, c1)
    P = W.grid_points(W.GridSpec(*g))
    _, cb = gwn.query_batch(m, torch.from_numpy(P).cuda(), want_chi=True)
    assert torch.equal(c1, cb)
    off = np.abs((w1.double() - w0.double()).cpu().numpy())
    pick = np.random.default_rng(1).choice(P.shape[0], min(1500, P.shape[0]), replace=False)
    perm = {"z": [0, 1, 2], "x": [1, 2, 0], "y": [2, 0, 1]}[axis]
    compare(w1.cpu().numpy()[pick], c1.cpu().numpy()[pick], s.V[:, perm], s.F, P[pick][:, perm],
            TOL_FP32 if prec == "fp32" else TOL_FP64, soup)
    from tests._util import off_surface_mask
    assert off[pick][off_surface_mask(s.V, s.F, P[pick])].max() <= SAME[prec]


@pytest.mark.parametrize("n_sheets", [20, 70])
def test_columns_with_many_crossings(gwn, n_sheets):
    # 70 stacked sheets: more crossings per column than a list holds
    s = W.wavy_sheets(n_sheets=n_sheets, n=12)
    m = _mesh(gwn, s.V, s.F)
    g = _grid(s.V, (23, 24, 90))
    w, c = gwn.query_grid(m, *g, want_chi=True)
    P = W.grid_points(W.GridSpec(*g))
    wb, cb = gwn.query_batch(m, torch.from_numpy(P).cuda(), want_chi=True)
    assert torch.equal(c, cb) and int(c.abs().max()) >= n_sheets - 1


def test_lists_of_few_large_triangles(gwn):
    # two triangles over every column (stripes), and one column at a time
    V = np.array([[-1, -1, 0.1], [1, -1, 0.0], [1, 1, -0.1], [-1, 1, 0.05]], np.float32)
    F = np.array([[0, 1, 2], [0, 2, 3]], np.int32)
    m = _mesh(gwn, V, F)
    for dims in ((200, 170, 9), (1, 1, 300), (1, 90, 1)):
        g = ((-1.1, -1.1, -0.5), tuple(2.2 / d for d in dims[:2]) + (1.0 / dims[2],), dims)
        w, c = gwn.query_grid(m, *g, want_chi=True)
        P = W.grid_points(W.GridSpec(*g))
        _, cb = gwn.query_batch(m, torch.from_numpy(P).cuda(), want_chi=True)
        assert torch.equal(c, cb)


def test_capture_takes_the_sum_over_all_chunks(gwn, monkeypatch):
    s = SOUPS["spheres"]()
    m = _mesh(gwn, s.V, s.F)
    g = _grid(s.V, (40, 40, 64))
    monkeypatch.setenv("GWN_GRID_FAR", "8")
    w1 = gwn.query_grid(m, *g)
    out = torch.empty_like(w1)
    st = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=st):
        gwn.query_grid(m, *g, out=out, stream=st)
    monkeypatch.setenv("GWN_GRID_FAR", "0")
    ref = gwn.query_grid(m, *g)
    for _ in range(3):
        out.fill_(-3.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert (out - ref).abs().max().item() <= SAME["fp32"]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("soup,dims,block,axis,flip", [
    ("spheres", (40, 33, 65), 8, "z", (1, 1, 1)),
    ("torus", (64, 1, 64), 8, "y", (1, 1, 1)),
    ("ellipsoids", (33, 9, 50), 8, "x", (-1, 1, -1)),
    ("fans", (20, 29, 257), 10, "z", (1, -1, 1)),
])
def test_gradient_far_part_equals_all_chunks(gwn, monkeypatch, prec, soup, dims, block, axis, flip):
    # the gradient's own bar against the oracle: relative to the sum of its edge terms' norms
    s = SOUPS[soup]()
    m = _mesh(gwn, s.V, s.F, axis=axis)
    g = _grid(s.V, dims, flip)
    monkeypatch.setenv("GWN_GRID_FAR", "0")
    g0 = gwn.query_grid_gradient(m, *g, prec=prec)
    monkeypatch.setenv("GWN_GRID_FAR", str(block))
    g1 = gwn.query_grid_gradient(m, *g, prec=prec)
    assert torch.equal(gwn.query_grid_gradient(m, *g, prec=prec), g1)
    P = W.grid_points(W.GridSpec(*g))
    pick = np.random.default_rng(2).choice(P.shape[0], min(1000, P.shape[0]), replace=False)
    ref, l1 = O.gradient(s.V, s.F, P[pick], axis=np.eye(3)[{"z": 2, "x": 0, "y": 1}[axis]], with_l1=True)
    ok = np.isfinite(ref).all(1) & np.isfinite(l1)
    bound = (2e-5 if prec == "fp32" else 1e-10) * np.maximum(1.0, l1[ok])[:, None]
    for got in (g0, g1):
        assert (np.abs(got.double().cpu().numpy()[pick][ok] - ref[ok]) <= bound).all()
    assert (np.abs((g1 - g0).double().cpu().numpy()[pick][ok]) <= bound).all()
