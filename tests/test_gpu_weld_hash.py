"""Welding sorts vertices by a 32-bit hash of their position: different positions of one hash, whose
vertices alternate in the input, stay apart, and each goes to the first vertex at its position."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _hash(P):
    """the hash as the library forms it (+0 and -0 alike)"""
    with np.errstate(over="ignore"):
        b = P.astype(np.float32).view(np.uint32).astype(np.uint64)
        b[(b & np.uint64(0x7fffffff)) == 0] = 0
        h = (b[:, 0] << np.uint64(32)) | b[:, 1]
        h = (h ^ (h >> np.uint64(33))) * np.uint64(0xff51afd7ed558ccd)
        h ^= b[:, 2] * np.uint64(0x9e3779b97f4a7c15)
        h = (h ^ (h >> np.uint64(33))) * np.uint64(0xc4ceb9fe1a85ec53)
        return (h >> np.uint64(32)).astype(np.uint32)


def test_positions_of_one_hash(gwn):
    rng = np.random.default_rng(3)
    P = np.unique(rng.uniform(-1, 1, (500_000, 3)).astype(np.float32), axis=0)
    h = _hash(P)
    order = np.argsort(h, kind="stable")
    same = np.flatnonzero(h[order][1:] == h[order][:-1])
    assert len(same) >= 10
    pairs = np.stack([order[same], order[same + 1]], 1)
    # triangles at both positions of each pair in turn, A B A B ..., and B A B A ... for every other
    V = []
    for k, (a, b) in enumerate(pairs):
        for i in range(6):
            corner = P[a] if (i + k) % 2 == 0 else P[b]
            V += [corner, *rng.uniform(-1, 1, (2, 3)).astype(np.float32)]
    V = np.array(V, np.float32)
    F = np.arange(len(V), dtype=np.int32).reshape(-1, 3)
    m = gwn.Mesh(torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda(), weld=True)
    i = m.info()
    unique = len(np.unique(V, axis=0))
    assert i["nunique"] == unique == len(V) - 4 * len(pairs)
    Fw, n = O.weld(V, F)
    assert n == unique and i["nboundary"] == len(O.boundary(Fw)[0])
    Q = rng.uniform(-1, 1, (5000, 3)).astype(np.float32)
    plain = gwn.Mesh(torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda())
    (w, c), (w0, c0) = (gwn.query_batch(x, torch.from_numpy(Q).cuda(), want_chi=True) for x in (m, plain))
    assert torch.equal(c, c0) and float((w - w0).abs().max()) <= 1e-5
