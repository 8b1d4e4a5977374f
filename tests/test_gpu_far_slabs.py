"""Grids over a small part of their mesh, with one coarse axis, so that boundary lies beyond the
grid's ends at the distance from which a level of the far part takes it: ribbons every half
step around that distance, beyond the last (ragged) block and before the first.  Against the
sum over all chunks and the gradient's oracle, with the bounds of the other far-part tests: the
interpolation's 2e-7 (FP32) and 6e-13 (FP64) of the nearest far terms and rounding in another
order.  A chunk counted twice or not at all is 1e-3 in w."""
import numpy as np
import pytest

import oracle as O

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SAME = {"fp32": 1e-5, "fp64": 1e-11}
STEP = {"x": (4.45, 1.0, 29.7), "y": (1.0, 4.45, 29.7)}
DIMS = {"x": (149, 200, 24), "y": (200, 149, 24)}


def _slab(axis, flip):
    """(V, F), origin, spacing, dims; lengths in units of the finest step, times 2^-7"""
    a = "xy".index(axis)
    step, dims = np.array(STEP[axis]), DIMS[axis]
    n, coarse = dims[a], step[a]
    V, F = [], []
    # around 2.5 and 3 half widths of the z axis' 24 samples: 185 to 245 coarse steps
    for side in (1, -1):
        for d in np.arange(185.0, 245.0, 0.5):
            x0 = (n - 0.5 + d) * coarse if side > 0 else (0.5 - d) * coarse
            t = np.linspace(0.0, 200.0, 29)
            p = np.zeros((2, 29, 3))
            p[:, :, a] = x0 + np.array([0.0, 3.0 * coarse])[:, None] * side
            p[:, :, 1 - a] = t
            p[:, :, 2] = 350.0 + 40.0 * np.sin(0.05 * t + d)
            b = len(V) * 58
            i = np.arange(28)
            F += [np.stack([b + i, b + i + 1, b + 29 + i], 1), np.stack([b + i + 1, b + 30 + i, b + 29 + i], 1)]
            V.append(p.reshape(-1, 3))
    k = sum(len(v) for v in V)
    V.append(np.array([[c * 4000.0 + e, c * 4000.0 + f, 300.0] for c in (-1, 1) for e, f in ((0, 0), (9, 0), (0, 9))]))
    F.append(np.array([[k, k + 1, k + 2], [k + 3, k + 4, k + 5]]))
    V = (np.concatenate(V) / 128).astype(np.float32)
    step = step / 128
    sp = step * np.array(flip)
    o = np.where(np.array(flip) > 0, 0.0, step * dims)
    return V, np.concatenate(F).astype(np.int32), tuple(o), tuple(sp), dims


def _mesh(gwn, V, F):
    return gwn.Mesh(torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda())


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("axis,flip", [("x", (1, 1, 1)), ("x", (-1, 1, 1)), ("y", (1, 1, 1)), ("y", (1, -1, -1))])
def test_chunks_past_the_ends(gwn, monkeypatch, prec, axis, flip):
    V, F, o, sp, dims = _slab(axis, flip)
    m = _mesh(gwn, V, F)
    monkeypatch.setenv("GWN_GRID_FAR", "0")
    w0 = gwn.query_grid(m, o, sp, dims, prec=prec)
    monkeypatch.setenv("GWN_GRID_FAR", "96")
    w1 = gwn.query_grid(m, o, sp, dims, prec=prec)
    assert not torch.equal(w0, w1)   # the far part was on
    assert float((w1 - w0).abs().max()) <= SAME[prec]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("axis,flip", [("x", (1, 1, 1)), ("y", (1, -1, 1))])
def test_gradient_past_the_ends(gwn, monkeypatch, prec, axis, flip):
    V, F, o, sp, dims = _slab(axis, flip)
    m = _mesh(gwn, V, F)
    monkeypatch.setenv("GWN_GRID_FAR", "96")
    g = gwn.query_grid_gradient(m, o, sp, dims, prec=prec)
    P = W.grid_points(W.GridSpec(o, sp, dims))
    # the last and the first blocks along the coarse axis, and anywhere
    a = "xy".index(axis)
    order = np.argsort(P[:, a], kind="stable")
    rng = np.random.default_rng(3)
    pick = np.concatenate([rng.choice(order[-90000:], 250), rng.choice(order[:90000], 250), rng.choice(len(P), 250)])
    ref, l1 = O.gradient(V, F, P[pick], axis=np.eye(3)[2], with_l1=True)
    ok = np.isfinite(ref).all(1) & np.isfinite(l1)
    got = g.double().cpu().numpy().reshape(-1, 3)[pick]
    bound = (2e-5 if prec == "fp32" else 1e-10) * np.maximum(1.0, l1[ok])[:, None]
    assert ok.sum() > 600
    assert (np.abs(got[ok] - ref[ok]) <= bound).all()
