"""A walk, and an export of per-leaf lists, that was refused memory leaves nothing
held, however often; the next one, with memory, is as the first."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import _say, compare_lists
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


# (the second: lists past the narrow slabs, whose exact storage is refused last)
@pytest.mark.parametrize("n,nll,theta,hs", [(9000, 8, 0.6, 1.0), (9000, 4, 0.0, 0.5)])
def test_refused(n, nll, theta, hs, monkeypatch):
    from paper_1108_0028_amd import RcbError
    _say("refused walk", n, nll, theta)
    c = W.small_random(n, 7000 + n, "uniform", h_scale=hs)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(theta)
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=nll, theta=theta)
    cells = 1 << t.info()["k"]
    ng = cells // 8
    lim.sizes.add(8 * ng * min(16384, cells))
    rooms = [0, 40 * ng, 4096 * ng, 40 * ng]
    if theta == 0.0:
        rooms.append(8 * ng * (1024 + 16384) + 200 * ng + 65536)
    # (32 bytes a group are the tree's own for all its walks)
    held = lim.live + 32 * ng + 4096
    for room in rooms:
        lim.budget = held + room
        with pytest.raises(RcbError) as e:
            t.walk()
        assert e.value.status == 2 and lim.live <= held
    lim.budget = 1 << 62
    t.walk()
    held = lim.live
    for room in (0, 16 * cells, 40 * cells):
        lim.budget = held + room
        with pytest.raises(RcbError) as e:
            t.export("near_off")
        assert e.value.status == 2 and lim.live <= held
        held = lim.live
    lim.budget = 1 << 62
    compare_lists(t, ot)
    t.destroy()
    assert lim.live == 0
