"""Mesh build where its forms meet: few boundary edges and loops in one workgroup or many
launches (8,192 edges, 2,048 loops), edge keys of as many bits as the vertices need, and
welding by hashed positions.  Against the direct sum over triangles (FP64, tolerance 1e-9:
both are sums of a few thousand FP64 terms of fixed-point positions, 2^-30 of the box) and
against numpy's unique positions."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _triangles(n, size, seed):
    rng = np.random.default_rng(seed)
    V = (rng.uniform(-1, 1, (n, 1, 3)) + size * rng.standard_normal((n, 3, 3))).reshape(-1, 3)
    return V.astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(-1, 3)


def _strip(n):
    """one loop of 2 n + 2 edges around a ribbon of 2 n triangles"""
    x = np.linspace(-1, 1, n + 1)
    V = np.stack([np.repeat(x, 2), np.tile([0.0, 0.3], n + 1), np.repeat(0.2 * np.sin(5 * x), 2)], -1)
    a = 2 * np.arange(n)[:, None]
    F = np.concatenate([a + [0, 2, 1], a + [1, 2, 3]])
    return V.astype(np.float32), F.astype(np.int32)


@pytest.mark.parametrize("name,soup,edges,loops", [
    ("2047 loops", lambda: _triangles(2047, 0.03, 1), 6141, 2047),
    ("2048 loops", lambda: _triangles(2048, 0.03, 1), 6144, 2048),
    ("2049 loops", lambda: _triangles(2049, 0.03, 1), 6147, 2049),
    ("8190 edges", lambda: _triangles(2730, 0.03, 2), 8190, 2730),
    ("8193 edges", lambda: _triangles(2731, 0.03, 2), 8193, 2731),
    ("a loop of 8192", lambda: _strip(4095), 8192, 1),
    ("a loop of 8194", lambda: _strip(4096), 8194, 1),
    ("one triangle", lambda: _triangles(1, 0.5, 3), 3, 1),
])
def test_boundary_paths(gwn, name, soup, edges, loops):
    V, F = soup()
    m = gwn.Mesh(_dev(V), _dev(F))
    i = m.info()
    assert (i["nboundary"], i["nloops"]) == (edges, loops)
    Q = _dev(np.random.default_rng(9).uniform(-1.1, 1.1, (500, 3)).astype(np.float32))
    w, d = gwn.query_batch(m, Q, prec="fp64"), gwn.query_direct(m, Q, prec="fp64")
    far = torch.ones(len(Q), dtype=torch.bool, device=Q.device)   # 2^-30 moves a triangle's angle by that over its distance
    dist = torch.cdist(Q.double(), _dev(V).double()).min(1).values
    far &= dist > 0.02
    assert (w - d).abs()[far].max().item() < 2.0 ** -30 * 2.5 / 0.02 * 16


@pytest.mark.parametrize("nv", [2, 3, 255, 256, 257, 65536, 65537, 300_000])
def test_weld_by_position(gwn, nv):
    """few distinct positions among many vertices, with zeros of either sign"""
    rng = np.random.default_rng(nv)
    k = max(2, nv // 5)
    P = (np.round(rng.uniform(-1, 1, (k, 3)) * 32) / 32).astype(np.float32)
    P[: k // 2, 2] = 0.0
    V = P[rng.integers(0, k, nv)]
    V[::3][V[::3] == 0] = np.float32(-0.0)
    F = rng.integers(0, nv, (max(1, nv // 3), 3)).astype(np.int32)
    m = gwn.Mesh(_dev(V), _dev(F), weld=True)
    U, inv = np.unique(V + np.float32(0.0), axis=0, return_inverse=True)   # -0 + 0 = 0
    assert m.info()["nunique"] == len(U)
    r = gwn.Mesh(_dev(U), _dev(inv.reshape(-1)[F].astype(np.int32)))
    assert r.info()["nboundary"] == m.info()["nboundary"]
    Q = _dev(rng.uniform(-1.2, 1.2, (200, 3)).astype(np.float32))
    a, b = (gwn.query_crossings(x, Q) for x in (m, r))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
