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


def _oracle_lists(c, nll):
    from oracle import oracle as O
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.7)
    off, ids, _ = ot.neighbours()
    return off, ids


@pytest.mark.parametrize("n,kind,hs", [(20000, "plummer", 1.0), (40000, "clumpy", 1.0), (3000, "uniform", 40.0)])
def test_smallest_scratch(n, kind, hs, monkeypatch):
    """the rows and the N/8 chunks are enough for a count: the lists that find no
    chunk are searched again by the fill call"""
    _say("smallest neighbour scratch", n, kind)
    c = W.clumpy_cube(n) if kind == "clumpy" else W.small_random(n, 11 + n, kind, h_scale=hs)
    off, ids = _oracle_lists(c, 12)
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=12, theta=0.7)
    t.walk()
    # row, head; pool of n / 8 + 1 chunks with 16 bytes each of bookkeeping; a word
    # per cell; the scan of the counts
    lim.budget = lim.live + 260 * n + 272 * (n // 8 + 1) + 4 * (1 << t.info()["k"]) + 8 * (n // 2048 + 1) + 256
    got = t.neighbours_count(_t(np.zeros(n + 1, np.int64)))
    assert lim.refused > 0 and got == len(ids)
    lim.budget = 1 << 62
    o, i = t.neighbours()
    np.testing.assert_array_equal(_np(o), off)
    np.testing.assert_array_equal(_np(i), ids)
    t.destroy()


def test_count_after_a_refused_count(monkeypatch):
    """a count without memory leaves nothing half made: the next one, with memory,
    is as the first"""
    from paper_1108_0028_amd import RcbError
    _say("count after a refused count")
    c = W.small_random(20000, 20011, "plummer")
    off, ids = _oracle_lists(c, 24)
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=24, theta=0.7)   # 1024 cells: no wide near slab to give back
    t.walk()
    live = lim.live
    for room in (0, 256 * c.n, 292 * c.n):   # (the smallest scratch takes 293 bytes a particle)
        lim.budget = live + room
        with pytest.raises(RcbError) as e:
            t.neighbours_count(_t(np.zeros(c.n + 1, np.int64)))
        assert e.value.status == 2 and lim.live == live
    lim.budget = 1 << 62
    o, i = t.neighbours()
    np.testing.assert_array_equal(_np(o), off)
    np.testing.assert_array_equal(_np(i), ids)
    t.destroy()
