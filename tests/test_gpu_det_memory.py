"""Deterministic VJP with little memory: the rows of source terms per 64 sink groups
are replaced by one row a particle where they cannot be had. The gradients meet the
bars of the deterministic form and repeat bit for bit."""
import numpy as np
import pytest

import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import _say
from test_gpu_vjp import TOL, _np, _t

pytestmark = pytest.mark.gpu


def _measured(monkeypatch, arrs, g, **options):
    """gradients, and the VJP's peak of workspace, with nothing refused"""
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, arrs, deterministic=True, **options)
    t.walk()
    t.gravity()
    held = lim.peak = lim.live
    out = t.vjp(*g)
    need = lim.peak - held
    t.destroy()
    return out, need


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_one_row_a_particle(prec, monkeypatch):
    import torch
    _say("deterministic vjp: one row a particle", prec)
    n = 20000
    c = W.small_random(n, 61, "uniform", h_scale=0.3)
    arrs = [_t(a) for a in c.arrays()]
    g = [_t(v, torch.float32 if prec == "mixed" else torch.float64) for v in W.cotangents(n, seed=4)]
    # theta = 0: each of the 8192 cells is near to all 1024 groups, 16 chunks of them
    opt = dict(n_ll=4, theta=0.0, precision=prec)
    ref, need = _measured(monkeypatch, arrs, g, **opt)
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, arrs, deterministic=True, **opt)
    t.walk()
    t.gravity()
    lim.budget = lim.live + need - (1 << 20)   # (of 10.2 MB for the rows of all chunks)
    one = t.vjp(*g)
    assert lim.refused > 0
    for a, b, r in zip(one, t.vjp(*g), ref):
        assert torch.equal(a, b)
        assert np.abs(_np(a) - _np(r)).max() <= TOL[prec] * np.abs(_np(r)).max()
    t.destroy()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_any_budget_above_the_least(prec, monkeypatch):
    """more memory than the form that recomputes node adjoints takes is never too
    little, however much of it the stored adjoints would leave"""
    import torch
    _say("deterministic vjp: budgets", prec)
    n = 12000
    c = W.small_random(n, 62, "plummer")
    arrs = [_t(a) for a in c.arrays()]
    g = [_t(v, torch.float32 if prec == "mixed" else torch.float64) for v in W.cotangents(n, seed=6)]
    opt = dict(n_ll=12, theta=0.6, precision=prec)
    ref, most = _measured(monkeypatch, arrs, g, **opt)
    with monkeypatch.context() as mp:
        mp.setenv("RCB_VJP_DET_RECOMPUTE", "1")
        _, least = _measured(mp, arrs, g, **opt)
    assert least < most
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, arrs, deterministic=True, **opt)
    t.walk()
    t.gravity()
    held = lim.live
    for i in range(33):
        lim.budget = held + least + (most - least) * i // 32
        for a, r in zip(t.vjp(*g), ref):
            assert np.abs(_np(a) - _np(r)).max() <= TOL[prec] * np.abs(_np(r)).max()
    t.destroy()
