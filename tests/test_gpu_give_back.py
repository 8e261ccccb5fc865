"""A call that lacks memory gives back what the tree holds beyond its need -- the
wide near slab for lists of their exact size, the neighbour pool for one of the chunks
in use -- and is made again. Results are those of a tree with memory, bit for bit:
the call's own, and those of a fill from the moved chunks."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import _np, _say, compare_lists
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu

CASES = [(20000, 8, "plummer", 1.0), (37013, 12, "clumpy", 1.0), (3000, 6, "uniform", 40.0)]


def _cloud(n, kind, hs):
    return W.clumpy_cube(n) if kind == "clumpy" else W.small_random(n, 11 + n, kind, h_scale=hs)


def _tree(lim, monkeypatch, arrs, nll, prec):
    return lim.tree(monkeypatch, arrs, n_ll=nll, theta=0.6, precision=prec, deterministic=True)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,nll,kind,hs", CASES[:2])   # (the third's pool is full, its near slab narrow)
def test_vjp_between_count_and_fill(n, nll, kind, hs, prec, monkeypatch):
    import torch
    _say("give back: vjp", n, kind, prec)
    c = _cloud(n, kind, hs)
    arrs = [_t(a) for a in c.arrays()]
    g = [_t(v, torch.float32 if prec == "mixed" else torch.float64) for v in W.cotangents(n, seed=9)]
    runs = []
    # (the stored adjoints are not taken: they are what a VJP does without first)
    monkeypatch.setenv("RCB_VJP_DET_RECOMPUTE", "1")
    for limited in (False, True):
        lim = LimitedAlloc()
        t = _tree(lim, monkeypatch, arrs, nll, prec)
        off = _t(np.zeros(n + 1, np.int64))
        total = t.neighbours_count(off)
        t.gravity()
        held = lim.peak = lim.live
        if limited:
            lim.budget = held + need // 2
        grad = t.vjp(*g)
        need = lim.peak - held
        print(f"   held {held}, needed {need}, held after {lim.live}", flush=True)
        if limited:
            assert lim.refused > 0 and lim.live < held - (1 << 20)
        lim.budget = lim.live + (64 << 10)
        ids = torch.full((total,), -1, dtype=torch.int32, device="cuda")
        t.neighbours_fill(off, ids)
        lim.budget = 1 << 62
        again = t.neighbours()
        acc = t.gravity()
        runs.append([*grad, *acc, off, ids, *again])
        t.destroy()
        assert lim.live == 0
    for a, b in zip(*runs):
        assert torch.equal(a, b)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.6)
    ooff, oids, _ = ot.neighbours()
    np.testing.assert_array_equal(_np(runs[1][-2]), ooff)
    np.testing.assert_array_equal(_np(runs[1][-1]), oids)


@pytest.mark.parametrize("n,nll,kind,hs", CASES)
def test_lists_kept_across_a_refresh(n, nll, kind, hs, monkeypatch):
    """a refresh on kept lists has no count to fill from: the neighbour scratch goes
    as a whole, and a new walk makes it again"""
    _say("give back: refresh", n, kind)
    c = _cloud(n, kind, hs)
    arrs = [_t(a) for a in c.arrays()]
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.6)
    lim = LimitedAlloc()
    t = _tree(lim, monkeypatch, arrs, nll, "fp64")
    ref = [a.clone() for a in t.gravity()]
    t.neighbours()
    t.refresh(*arrs, keep_lists=True)
    held = lim.live
    lim.budget = held
    t.refresh(*arrs, keep_lists=True)
    assert lim.refused > 0 and lim.live < held - 260 * n
    lim.budget = 1 << 62
    for a, b in zip(t.gravity(), ref):
        assert bool((a == b).all())
    compare_lists(t, ot)
    t.walk()
    ooff, oids, _ = ot.neighbours()
    off, ids = t.neighbours()
    np.testing.assert_array_equal(_np(off), ooff)
    np.testing.assert_array_equal(_np(ids), oids)
    t.destroy()
