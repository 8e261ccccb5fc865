"""The overflow pool of the neighbour search is sized by the walk's estimate of the
lists' lengths, by the particles' spread over the axes that a cloud has and in any
unit of length: the scratch of a planar or linear cloud of 50 neighbours stays near
that of a cloud with volume, and its lists are those of the all-pairs search."""
import numpy as np
import pytest

from oracle import brute
import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import _np, _say
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


def _cloud(dims, n, unit=1.0):
    """n particles uniform in `dims` axes of the unit cube, h for 50 neighbours"""
    rng = np.random.default_rng(77)
    x = [rng.uniform(0.0, 1.0, n) if d < dims else np.full(n, 0.3) for d in range(3)]
    r = {1: 25.0 / n, 2: np.sqrt(50.0 / (np.pi * n)), 3: (50.0 / (4.19 * n)) ** (1 / 3)}[dims]
    return W.Cloud("flat", *[v * unit for v in x], np.full(n, 1.0 / n), np.full(n, 0.5 * r * unit))


def _search(c, monkeypatch):
    """(offsets, ids, scratch bytes of the count call)"""
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=12, theta=0.7)
    t.walk()
    before = lim.live
    off, ids = t.neighbours()
    held = lim.live - before
    t.destroy()
    assert lim.live == 0
    return _np(off), _np(ids), held


@pytest.mark.parametrize("dims", [1, 2])
def test_flat_clouds(dims, monkeypatch):
    _say("pool of a flat cloud", dims)
    c = _cloud(dims, 12000)
    off, ids, _ = _search(c, monkeypatch)
    boff, bids = brute.neighbours(c.x, c.y, c.z, c.h)
    np.testing.assert_array_equal(off, boff)
    np.testing.assert_array_equal(ids, bids)
    # (past the sizes that get the longest lists' pool whatever the estimate)
    n = 400_000
    _, _, flat = _search(_cloud(dims, n), monkeypatch)
    _, _, full = _search(_cloud(3, n), monkeypatch)
    print(f"   scratch per particle: {flat / n:.0f} B, with volume {full / n:.0f} B", flush=True)
    # row 256, heads and queues 5, pool N/8 chunks 33; the estimates differ by the
    # ratio of 4.19 to pi, or 2, and by the cells' scatter: two chunks a particle
    assert flat <= full + 2 * 260 * n


@pytest.mark.parametrize("log2s", [-400, 400])
def test_units(log2s, monkeypatch):
    """lengths whose cube is past the range"""
    _say("pool in units of 2 **", log2s)
    n = 400_000
    off, ids, held = _search(_cloud(3, n), monkeypatch)
    soff, sids, sheld = _search(_cloud(3, n, 2.0 ** log2s), monkeypatch)
    np.testing.assert_array_equal(soff, off)
    np.testing.assert_array_equal(sids, ids)
    assert sheld == held
