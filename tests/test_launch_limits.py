"""Launches whose size goes with the call's stay below the 2^32 work-items that a launch can
have (host code, no GPU)."""
import ctypes

import pytest

from paper_2605_01536_amd import gwn


@pytest.mark.parametrize("kernel", [0, 1, 2])
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
