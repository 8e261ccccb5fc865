"""Gravity with the wave counts per group of cells that its launch chooses
from the number of groups: the forces (and small clouds' VJP) match the oracle at cell
counts on each side of the limits, with cells of 1 to a few hundred particles
(the last of them sinks in several passes, the last pass ragged)."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from test_gpu_parity import TOL, _gpu_tree, _np, _say, gate
from test_gpu_vjp import TOL as VTOL, _t

pytestmark = pytest.mark.gpu


# 1024 and 2048 groups of 8 cells (8192 / 16384 cells); one group of 1, 2, 4 cells
@pytest.mark.parametrize("n,nll", [(16000, 2), (20000, 2), (90, 100), (90, 50), (300, 90)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_forces_at_group_counts(n, nll, prec):
    import torch
    c = W.small_random(n, 90 + n, "uniform", h_scale=0.2 if n < 1000 else 0.02)
    if n > 1000:   # one cell of 333 particles: five passes of 64 sinks and one of 13
        c.x[:333], c.y[:333], c.z[:333] = 0.3, 0.2, 0.1
    _say("group waves", n, nll, prec)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.9)
    ref = np.stack(ot.gravity(), 1)
    gt = _gpu_tree(c, nll, 0.9, prec)
    a = np.stack([_np(v).astype(np.float64) for v in gt.gravity()], 1)
    assert gate(a, ref) <= (1e-11 if prec == "fp64" else TOL[prec])
    if n > 1000:
        gt.destroy()
        return
    g = W.cotangents(c.n, seed=3)
    vref = ot.vjp(*g)
    dt = torch.float32 if prec == "mixed" else torch.float64
    for x, r in zip(gt.vjp(*[_t(v, dt) for v in g]), vref):
        assert np.abs(_np(x).astype(np.float64) - r).max() <= VTOL[prec] * np.abs(r).max()
    gt.destroy()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_deterministic_source_chunks(prec):
    """theta = 0: every cell is near to all 256 groups, so its source-side
    terms come from several chunks of sink groups; one cell of 200 particles."""
    import torch
    from paper_1108_0028_amd import Tree
    c = W.small_random(3000, 31, "plummer", h_scale=0.5)
    c.x[:200], c.y[:200], c.z[:200] = 0.3, 0.2, 0.1
    _say("source chunks", prec)
    ot = O.OracleTree(*c.arrays(), n_ll=2)
    ot.walk(0.0)
    g = W.cotangents(c.n, seed=4)
    vref = ot.vjp(*g)
    dt = torch.float32 if prec == "mixed" else torch.float64
    gt = Tree(*[_t(v) for v in c.arrays()], n_ll=2, theta=0.0, precision=prec, deterministic=True)
    first = gt.vjp(*[_t(v, dt) for v in g])
    for x, y, r in zip(first, gt.vjp(*[_t(v, dt) for v in g]), vref):
        assert torch.equal(x, y)
        assert np.abs(_np(x).astype(np.float64) - r).max() <= VTOL[prec] * np.abs(r).max()
    gt.destroy()
