"""Near slabs of 1024 entries per group where the wider ones cannot be had: lists
longer than they are go through the exact second walk, in both walk modes, and a
workspace that holds them is enough for a walk. Lists, neighbours and forces are
the oracle's."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import TOL, _np, _say, compare_lists, gate
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pure", [False, True])
@pytest.mark.parametrize("n,nll,kind,hs,theta", [(9000, 6, "clustered", 40.0, 0.6),   # every cell a candidate
                                                 (9000, 4, "uniform", 0.5, 0.0)])     # every cell near
def test_lists_past_the_narrow_slabs(n, nll, kind, hs, theta, pure, monkeypatch):
    c = W.small_random(n, 7000 + n, kind, h_scale=hs)
    _say("lists past the narrow slabs", n, nll, kind, theta, pure)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(theta, pure_mac=pure)
    ref = np.stack(ot.gravity(), 1)
    ooff, oids, _ = ot.neighbours()
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=nll, theta=theta, pure_mac=pure)
    leaves = 1 << t.info()["k"]
    lim.sizes.add(8 * (leaves // 8) * min(16384, leaves))
    t.walk()
    assert lim.refused == 1
    compare_lists(t, ot)
    assert int(np.diff(_np(t.export("near_off"))).max()) > 1024
    off, ids = t.neighbours()
    np.testing.assert_array_equal(_np(off), ooff)
    np.testing.assert_array_equal(_np(ids), oids)
    assert gate(np.stack([_np(a) for a in t.gravity()], 1), ref) < TOL["fp64"]
    t.destroy()


def test_workspace_of_the_narrow_slabs(monkeypatch):
    c = W.small_random(20000, 27000, "uniform", h_scale=0.5)
    _say("workspace of the narrow slabs", c.n)
    ot = O.OracleTree(*c.arrays(), n_ll=8)
    ot.walk(0.6)
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=8, theta=0.6)
    ng = (1 << t.info()["k"]) // 8
    # the slabs, and per group 16 bytes of counts, 16 of queues and statistics, 32
    # of list ends
    lim.budget = lim.live + 8 * ng * (1024 + 16384) + 64 * ng + 4096
    t.walk()
    assert lim.refused == 1
    lim.budget = 1 << 62
    compare_lists(t, ot)
    t.destroy()
