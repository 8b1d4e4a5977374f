"""Launches whose size goes with the call's stay below the 2^32 work-items that a launch can
have (host code, no GPU)."""
import ctypes

import pytest

from paper_2605_01536_amd import gwn


@pytest.mark.parametrize("kernel", [0, 1, 2, 3])
@pytest.mark.parametrize("limit", [None, "256"])
def test_plan_kernels(monkeypatch, kernel, limit):
    if limit:
        monkeypatch.setenv("GWN_MAX_LAUNCH_QUERIES", limit)
    f = gwn.load().gwn_test_plan_launches
    f.restype = ctypes.c_int64
    w = ctypes.c_int64()
    # 2^31 queries in items of 128 and of 64, 2^33 in items of 128
    for n in (1, 5, 1 << 24, 1 << 25, 1 << 26) if not limit else (1, 5, 4097):
        launches = f(ctypes.c_int64(n), ctypes.c_int32(kernel), ctypes.byref(w))
        assert launches >= 1 and w.value < 1 << 32
        assert limit is None or w.value <= 1024   # one item


@pytest.mark.parametrize("n", [64, 645, 646, 1020, 1021, 1024])
def test_boxes_of_samples(monkeypatch, n):
    # an unwelded soup of 333,000 triangles: as many loops of three edges
    d = lambda *x: (ctypes.c_double * len(x))(*x)
    f = gwn.load().gwn_test_boxes
    f.restype = ctypes.c_int64
    w = ctypes.c_int64()

    def boxes():
        return f(d(0, 0, 0, 1, 1, 1), ctypes.c_int64(167_000), ctypes.c_double(1e6), ctypes.c_int64(999_000),
                 ctypes.c_int64(333_000), ctypes.c_int64(33_300), d(0, 0, 0), d(1 / n, 1 / n, 1 / n),
                 (ctypes.c_int64 * 3)(n, n, n), ctypes.byref(w))
    b = boxes()
    assert b * 64 >= n ** 3 and w.value < 1 << 32   # in boxes, and every launch is one that can be made
    if n == 64:
        monkeypatch.setenv("GWN_MAX_LAUNCH_QUERIES", "1024")
        assert boxes() == b and w.value <= 1024
