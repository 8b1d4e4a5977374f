"""The gradient next to a boundary vertex at the origin, where floats are fine enough for distances
whose fourth power leaves FP32's range (from about 1e-18 of the mesh's size): finite, and against the
boundary's Biot-Savart sum in FP64.  A term is rounded some ten times, hence 1e-6 (FP32) and 1e-13."""
import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

V = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1], [1, 1, 1]], np.float32)
F = np.array([[0, 1, 2], [0, 2, 3], [1, 4, 2]], np.int32)
EDGES = [(0, 1), (1, 4), (4, 2), (2, 3), (3, 0)]


def _exact(Q):
    out = np.zeros((len(Q), 3))
    for a, b in EDGES:
        A, B = V[a].astype(np.float64) - Q, V[b].astype(np.float64) - Q
        la, lb = np.linalg.norm(A, axis=1), np.linalg.norm(B, axis=1)
        den = la * lb * (la * lb + (A * B).sum(1))
        out += np.cross(A, (V[b] - V[a]).astype(np.float64)) * ((la + lb) / den)[:, None]
    return out / (4 * np.pi)


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-6), ("fp64", 1e-13)])
@pytest.mark.parametrize("axis", ["z", "x"])
def test_points_and_grids(gwn, prec, tol, axis):
    m = gwn.Mesh(torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda(), axis=axis)
    d = 10.0 ** -np.arange(3, 33.0, 0.5)
    Q = np.stack([0.7 * d, -0.5 * d, -0.31 * d], 1).astype(np.float32)
    ref = _exact(Q.astype(np.float64))
    for n in (len(Q), 1):
        g = gwn.query_gradient(m, torch.from_numpy(Q[-n:]).cuda(), prec=prec).double().cpu().numpy()
        assert (np.abs(g - ref[-n:]).max(1) <= tol * np.abs(ref[-n:]).max(1)).all()
    # and beside boundary enough for the kernels of long boundaries, far away
    for n_v in (1, 60):   # 1,200 edges or so, and over 4,096
        far = W.torus_soup(seed=3, n_u=40 + n_v, n_v=30 + n_v)
        U, G = np.concatenate([V, far.V + np.float32(30)]), np.concatenate([F, far.F + len(V)]).astype(np.int32)
        big = gwn.Mesh(torch.from_numpy(U).cuda(), torch.from_numpy(G).cuda(), axis=axis)
        g = gwn.query_gradient(big, torch.from_numpy(Q).cuda(), prec=prec).double().cpu().numpy()
        # (the torus adds less than its area over the cube of its distance)
        assert (np.abs(g - ref).max(1) <= tol * np.abs(ref).max(1) + 1e-3).all()
    for s in (1e-6, 1e-19, 1e-21, 1e-27):
        grid = ((0.0, 0.0, 0.0), (-s, -1.3 * s, -0.8 * s), (3, 2, 130))
        P = W.grid_points(W.GridSpec(*grid))
        ref_g = _exact(P.astype(np.float64))
        g = gwn.query_grid_gradient(m, *grid, prec=prec).double().cpu().numpy().reshape(-1, 3)
        assert (np.abs(g - ref_g).max(1) <= tol * np.abs(ref_g).max(1)).all(), s


# grids of columns enough for a wave each, one sample or two to a lane: on boundary enough the
# samples are taken again by a kernel of their own (also cut into launches)
@pytest.mark.parametrize("dims", [(64, 65, 3), (45, 31, 130)])
@pytest.mark.parametrize("axis", ["z", "x", "y"])
@pytest.mark.parametrize("launch", [None, "65536"])
def test_large_grids(gwn, monkeypatch, dims, axis, launch):
    if launch:
        monkeypatch.setenv("GWN_MAX_LAUNCH_QUERIES", launch)
    far = W.torus_soup(seed=3, n_u=41, n_v=31)
    U, G = np.concatenate([V, far.V + np.float32(30)]), np.concatenate([F, far.F + len(V)]).astype(np.int32)
    m = gwn.Mesh(torch.from_numpy(U).cuda(), torch.from_numpy(G).cuda(), axis=axis)
    assert m.info()["nboundary"] >= 512
    for s in (1e-6, 1e-21):
        grid = ((0.0, 0.0, 0.0), (-s, -1.3 * s, -0.8 * s), dims)
        ref = _exact(W.grid_points(W.GridSpec(*grid)).astype(np.float64))
        g = gwn.query_grid_gradient(m, *grid, prec="fp32").double().cpu().numpy().reshape(-1, 3)
        assert (np.abs(g - ref).max(1) <= 1e-6 * np.abs(ref).max(1) + 1e-3).all(), s
