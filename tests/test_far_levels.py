"""The levels of a grid's far part share out the boundary's chunks (host code, no GPU): for
every block of columns each chunk is summed exactly once, near the block or at one of the
levels, wherever it lies; also past the grid's end, for grids over a part of their mesh with
unequal steps, whose coarsest blocks are one step short of or beyond their children's."""
import ctypes

import numpy as np
import pytest

from paper_2605_01536_amd import gwn

QMAX = 2.0 ** 30 - 1


def _plan(bbox, nchunk, chunk_w, origin, spacing, dims, prec, values):
    L = gwn.load()
    f = L.gwn_test_far_plan
    f.restype = ctypes.c_int64
    out = np.zeros(1 << 20, np.int64)
    d = lambda x: (ctypes.c_double * len(x))(*x)
    n = f(d(bbox), ctypes.c_int64(nchunk), ctypes.c_double(chunk_w), d(origin), d(spacing),
          (ctypes.c_int64 * 3)(*dims), ctypes.c_int32(prec), ctypes.c_int32(values),
          out.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(out.size))
    assert n >= 1
    it = iter(out[:n].tolist())
    levels = []
    for _ in range(next(it)):
        thr, axes = next(it), []
        for _ in range(2):
            nc = next(it)
            axes.append(np.array([[next(it), next(it)] for _ in range(nc)]))
        levels.append((thr, axes))
    assert next(it, None) is None
    return levels


def _qgrid(bbox):
    """The fixed-point grid as the library lays it: 1.75 sizes around, a power of two of cells per unit."""
    lo, hi = np.array(bbox[:3]), np.array(bbox[3:])
    e = float((hi - lo).max())
    k = int(np.floor(np.log2(QMAX / (2.5 * e))))
    return lo - 0.75 * e, 2.0 ** k


def _ranges(levels, origin, spacing, glo, scale):
    """Quantised range of every block in x and y per level."""
    out = []
    for thr, axes in levels:
        r = []
        for a in range(2):
            x = (np.float64(origin[a]) + (axes[a] + 0.5) * np.float64(spacing[a])).astype(np.float32).astype(np.float64)
            q = np.rint((x - glo[a]) * scale)
            r.append(np.sort(q, axis=1))
        out.append((thr, r))
    return out


def _far(rng, thr, b, chunks):
    """(chunks,) far from the block b = (bx, by)"""
    d = [np.maximum(chunks[:, 2 * a] - rng[a][b[a]][1], rng[a][b[a]][0] - chunks[:, 2 * a + 1]) for a in range(2)]
    return np.maximum(d[0], d[1]) >= thr


def _count(levels, b, chunks):
    """How often each chunk is summed for the samples of level 0's block b."""
    n = np.zeros(len(chunks), int)
    far = []
    for l, (thr, r) in enumerate(levels):
        far.append(_far(r, thr, tuple(min(b[a] >> l, len(r[a]) - 1) for a in range(2)), chunks))
    n += ~far[0]
    for l in range(len(levels)):
        n += far[l] & ~(far[l + 1] if l + 1 < len(levels) else np.zeros(len(chunks), bool))
    return n


def _check(levels, origin, spacing, dims, bbox, rng):
    glo, scale = _qgrid(bbox)
    lv = _ranges(levels, origin, spacing, glo, scale)
    # boxes of chunks over the mesh, and some whose edge lies at the far distance from a block's end
    m = 3000
    c = np.empty((m, 4))
    for a in range(2):
        lo = (bbox[a] - glo[a]) * scale
        hi = (bbox[3 + a] - glo[a]) * scale
        c[:, 2 * a] = rng.uniform(lo, hi, m)
        step = abs(spacing[a]) * scale
        for j in range(0, m, 2):
            thr, r = lv[rng.integers(len(lv))]
            blk = r[a][rng.choice([0, len(r[a]) - 1])]
            up = rng.random() < 0.5
            edge = blk[1] + thr if up else blk[0] - thr
            edge += rng.uniform(-2.5, 2.5) * step
            c[j, 2 * a] = edge if up else edge - 0.3 * step
        c[:, 2 * a + 1] = c[:, 2 * a] + rng.uniform(0, 0.3, m) * step
    c = np.rint(c)
    n0 = [len(lv[0][1][a]) for a in range(2)]
    blocks = {(i, j) for i in (0, n0[0] - 1) for j in (0, n0[1] - 1)}
    blocks |= {(int(rng.integers(n0[0])), int(rng.integers(n0[1]))) for _ in range(6)}
    for b in blocks:
        n = _count(lv, b, c)
        assert (n == 1).all(), (b, np.unique(n), int((n != 1).sum()))


BOX = (0.0, 0.0, 0.0, 1.0, 1.0, 1.0)


@pytest.mark.parametrize("dims,steps,prec,values,nchunk", [
    ((14, 264, 16), (0.0212, 0.000643, 0.0099), 0, 1, 1533),
    ((149, 200, 24), (0.00267, 0.0006, 0.01782), 0, 1, 1533),
    ((200, 149, 24), (0.0006, 0.00267, 0.01782), 0, 3, 1533),
    ((160, 150, 20), (0.0006, 0.0021, 0.0153), 1, 1, 20000),
])
def test_named_layouts(dims, steps, prec, values, nchunk):
    # clipped coarsest blocks beside an axis whose eight coarse samples set the distance
    rng = np.random.default_rng(1)
    origin = (0.02, 0.02, 0.02)
    levels = _plan(BOX, nchunk, 2e5, origin, steps, dims, prec, values)
    assert levels
    _check(levels, origin, steps, dims, BOX, rng)


@pytest.mark.parametrize("seed", range(12))
def test_every_chunk_once(seed):
    rng = np.random.default_rng(seed)
    deep = 0
    for _ in range(60):
        dims = [int(np.exp(rng.uniform(0, np.log(500)))) for _ in range(3)]
        ratio = np.exp(rng.uniform(0, np.log(40), 3))
        if rng.random() < 0.5:   # one axis of few samples at coarse steps
            a = int(rng.integers(3))
            dims[a], ratio[a] = int(rng.integers(11, 30)), rng.uniform(20, 40)
        size = ratio * dims
        steps = ratio / size.max() * rng.uniform(0.05, 0.9)
        sign = rng.choice([1, 1, -1], 3)
        start = [rng.uniform(0, 1 - steps[a] * dims[a]) for a in range(3)]
        origin = tuple(float(start[a] if sign[a] > 0 else start[a] + steps[a] * dims[a]) for a in range(3))
        spacing = tuple(float(x) for x in steps * sign)
        prec, values = int(rng.integers(2)), int(rng.choice([1, 3]))
        levels = _plan(BOX, int(np.exp(rng.uniform(4, 11))), float(np.exp(rng.uniform(10, 18))), origin, spacing,
                       dims, prec, values)
        deep += len(levels) >= 2
        if levels:
            for (thr, lo), (up, hi) in zip(levels, levels[1:]):
                assert thr <= up   # the distances do not fall, and the blocks nest
                for a in range(2):
                    of = hi[a][np.minimum(np.arange(len(lo[a])) // 2, len(hi[a]) - 1)]
                    assert (lo[a][:, 0] >= of[:, 0]).all() and (lo[a][:, 1] <= of[:, 1]).all()
            _check(levels, origin, spacing, dims, BOX, rng)
    assert deep >= 3
