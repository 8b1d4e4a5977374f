"""Grids in boxes of samples (k_grid_boxes): every sample has the bits of a query at its position,
whatever the remainders of the box, the number of waves that share it, the ray axis, and where the
crossings come from (lists, a walk per sample: too many crossings in a column, falling coordinates,
a captured stream)."""
import numpy as np
import pytest
import torch

from paper_2605_01536_amd import gwn
from paper_2605_01536_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _positions(origin, spacing, dims):
    ax = [(np.float64(o) + (np.arange(n) + 0.5) * np.float64(s)).astype(np.float32)
          for o, s, n in zip(origin, spacing, dims)]
    return torch.from_numpy(np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)).cuda()


def _mesh(axis="z", n=4000):
    s = wl.ellipsoid_union(np.random.default_rng(5), n, 0.1)
    return s, gwn.build_mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda(), axis=axis)


def _check(mesh, origin, spacing, dims):
    w, chi = gwn.query_grid(mesh, origin, spacing, dims, prec="fp32", want_chi=True)
    rw, rchi = gwn.query_batch(mesh, _positions(origin, spacing, dims), prec="fp32", want_chi=True)
    assert torch.equal(chi.reshape(-1), rchi)
    assert torch.equal(w.reshape(-1), rw)
    return w


# boxes: 1, 1, 2 x 2 x 2, 125 and 256 (16 waves each), 260 and 1,024 (8), 1,040 and 1,560 (4)
@pytest.mark.parametrize("dims", [(1, 1, 1), (4, 4, 4), (5, 7, 8), (20, 20, 20), (32, 32, 13), (20, 49, 13),
                                  (64, 29, 31), (37, 50, 29), (3, 240, 101), (70, 1, 31), (1, 1, 100), (130, 90, 1)])
@pytest.mark.parametrize("axis", ["x", "y", "z"])
def test_bits_of_the_points(monkeypatch, dims, axis):
    monkeypatch.setenv("GWN_GRID_BOXES", "1")
    s, m = _mesh(axis)
    lo, hi = s.bbox()
    sp = tuple(float(x) for x in 1.1 * (hi - lo) / np.array(dims))
    _check(m, tuple(float(x) for x in lo - 0.05 * (hi - lo)), sp, dims)


def test_falling_coordinates_and_far_outside(monkeypatch):
    monkeypatch.setenv("GWN_GRID_BOXES", "1")
    s, m = _mesh()
    lo, hi = s.bbox()
    e = float((hi - lo).max())
    _check(m, tuple(float(x) for x in hi), (-e / 9, e / 11, -e / 10), (9, 8, 10))
    # half inside the fixed-point box, half up to 50 sizes away
    _check(m, tuple(float(x) for x in lo - 50 * e), (5.1 * e, 5.0 * e, 4.9 * e), (20, 21, 22))


def test_many_crossings_in_a_column(monkeypatch):
    monkeypatch.setenv("GWN_GRID_BOXES", "1")
    rng = np.random.default_rng(2)
    V, F = [], []
    for i in range(48):   # 48 sheets of 18 triangles, one hole each: up to 48 crossings
        g = np.linspace(-1, 1, 4)
        x, y = np.meshgrid(g, g, indexing="ij")
        v = np.stack([x, y, np.full_like(x, i / 48) + 0.004 * rng.uniform(size=x.shape)], -1).reshape(-1, 3)
        q = [(4 * a + b, 4 * a + b + 4, 4 * a + b + 5, 4 * a + b + 1) for a in range(3) for b in range(3)]
        f = [t for c in q for t in ((c[0], c[1], c[2]), (c[0], c[2], c[3]))]
        f.pop(int(rng.integers(len(f))))
        F += [[16 * i + k for k in t] for t in f]
        V.append(v)
    m = gwn.build_mesh(torch.from_numpy(np.concatenate(V).astype(np.float32)).cuda(),
                       torch.tensor(F, dtype=torch.int32).cuda())
    w = _check(m, (-1.1, -1.1, -0.2), (0.1, 0.1, 0.05), (22, 22, 26))
    assert float(w.max()) - float(w.min()) > 10


def test_captured(monkeypatch):
    monkeypatch.setenv("GWN_GRID_BOXES", "1")
    s, m = _mesh()
    lo, hi = s.bbox()
    args = (m, tuple(float(x) for x in lo), tuple(float(x) for x in (hi - lo) / 24), (24, 24, 24))
    ref = gwn.query_grid(*args, prec="fp32")
    out = torch.empty_like(ref)
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        gwn.query_grid(*args, prec="fp32", out=out)
    stream.synchronize()
    with torch.cuda.graph(g, stream=stream):
        gwn.query_grid(*args, prec="fp32", out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_chosen_by_the_time_of_either(monkeypatch):
    """Short loops and few samples take boxes (the points' bits); the choice of a column form does not."""
    s, m = _mesh(n=30000)
    lo, hi = s.bbox()
    o, sp, dims = tuple(float(x) for x in lo), tuple(float(x) for x in (hi - lo) / 40), (40, 40, 40)
    rw = gwn.query_batch(m, _positions(o, sp, dims), prec="fp32")
    assert torch.equal(gwn.query_grid(m, o, sp, dims, prec="fp32").reshape(-1), rw)
    monkeypatch.setenv("GWN_GRID_SAMPLES_PER_LANE", "1")
    w = gwn.query_grid(m, o, sp, dims, prec="fp32").reshape(-1)
    assert not torch.equal(w, rw)
    # both within 4e-6 of each other: an FP32 sum of some hundred near angles of one ulp each
    assert float((w - rw).abs().max()) < 4e-6
