"""Tuning lines that earlier kernels' timings left in a cache file are not used."""
import json

import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_lines_of_other_kernels(gwn, tmp_path, monkeypatch):
    for v in ("GWN_SPLIT_BOUNDARY", "GWN_ORDER_QUERIES", "GWN_GRID_SAMPLES_PER_LANE"):
        monkeypatch.delenv(v, raising=False)
    s = W.torus_soup(seed=3, n_u=40, n_v=30)
    V, F = torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda()
    m = gwn.Mesh(V, F)
    cache = tmp_path / "tune.jsonl"
    m.autotune("fp32", grid_nz=64, reps=1, cache=str(cache))
    line = json.loads(cache.read_text())
    old = dict(line, key=line["key"].replace("|mesh2|", "|mesh|"), split_max_points=77, order_min_points=-1)
    assert old["key"] != line["key"]
    cache.write_text(json.dumps(old) + "\n")
    assert gwn.Mesh(V, F).autotune("fp32", grid_nz=64, reps=1, cache=str(cache))["split_max_points"][0] != 77
    assert len(cache.read_text().splitlines()) == 2   # timed, and added
    Q = torch.from_numpy(np.concatenate([W.uniform_box(np.random.default_rng(1), 3000, *s.bbox())])).cuda()
    plans = tmp_path / "plans.jsonl"
    gwn.MultiPlan([m], Q, [0, 3000], autotune=True, tune_cache=str(plans))
    line = json.loads(plans.read_text())
    plans.write_text(json.dumps(dict(line, key=line["key"].replace("|plan2|", "|"), item_queries=192)) + "\n")
    p = gwn.MultiPlan([m], Q, [0, 3000], autotune=True, tune_cache=str(plans))
    assert p.info()["item_queries"] != 192 and len(plans.read_text().splitlines()) == 2
