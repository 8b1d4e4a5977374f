"""Calls whose orders of points are their own choice do without where the memory for them cannot
be had: the same results as with them."""
import ctypes

import numpy as np
import pytest

from paper_2605_01536_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture
def hook(gwn):
    f = gwn.load().gwn_test_fail_alloc_after
    f.argtypes = [ctypes.c_int64]
    f.restype = ctypes.c_int64
    f(-1)
    yield f
    f(-1)


def _case(gwn, n):
    s = W.torus_soup(seed=2, n_u=130, n_v=100)
    m = gwn.Mesh(torch.from_numpy(s.V).cuda(), torch.from_numpy(s.F).cuda())
    return m, torch.from_numpy(W.uniform_box(np.random.default_rng(3), n, *s.bbox())).cuda()


def test_batch(gwn, hook):
    m, Q = _case(gwn, 60_000)    # in order along a curve for the boundary sum, not for the crossings
    chi = torch.empty(len(Q), dtype=torch.int32, device="cuda")
    hook(-1)
    ref = gwn.query_batch(m, Q, want_chi=True, chi_out=chi)[0]
    assert hook(-1) == 2         # the order and its sort's scratch
    for k in (0, 1):
        hook(k)
        w = gwn.query_batch(m, Q, want_chi=True, chi_out=chi)[0]
        hook(-1)
        assert torch.equal(w, ref)


def test_plan(gwn, hook):
    m, Q = _case(gwn, 60_000)
    offs = [0, 20_000, 60_000]
    hook(-1)
    plan = gwn.MultiPlan([m, m], Q, offs)
    n = hook(-1)
    ref = plan.run().clone()
    served = 0
    for k in range(n):
        hook(k)
        try:
            plan = gwn.MultiPlan([m, m], Q, offs)
        except gwn.GwnError as e:
            assert e.status == 2
            plan = None
        hook(-1)
        if plan is not None:
            served += 1
            torch.cuda.synchronize()
            assert torch.equal(plan.run(), ref)
            plan.close()
    assert served == 4           # two orders with a sort's scratch each
