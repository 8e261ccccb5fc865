"""Staging of near-field sources: tiles of 64 whose entries are found by marks
at their starts. Cells of one particle (64 starts in a tile), of sizes around a
tile, empty cells between others (coincident particles), lists of more than one
chunk of 64 entries and of less than one tile; everything is near (theta = 0)."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from test_gpu_parity import TOL, _gpu_tree, _np, _say, gate
from test_gpu_vjp import TOL as VTOL, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nll", [(1, 1), (40, 1), (300, 1), (64, 64), (126, 63), (130, 65), (700, 90)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("coincident", [False, True])
def test_tiles(n, nll, prec, coincident):
    import torch
    _say("staging", n, nll, prec, coincident)
    c = W.small_random(n, 40 + n, "uniform", h_scale=1.0)
    if coincident:   # a third of the particles at one point: empty cells beside them
        c.x[:n // 3], c.y[:n // 3], c.z[:n // 3] = 0.3, 0.2, 0.1
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.0)
    gt = _gpu_tree(c, nll, 0.0, prec)
    off, ids, _ = ot.neighbours()
    goff, gids = gt.neighbours()
    assert np.array_equal(_np(goff), off) and np.array_equal(_np(gids), ids)
    a = np.stack([_np(v).astype(np.float64) for v in gt.gravity()], 1)
    ref = np.stack(ot.gravity(), 1)
    if n == 1:
        assert np.all(a == 0.0)
    else:
        assert gate(a, ref) <= (1e-11 if prec == "fp64" else TOL[prec])
        g = W.cotangents(n, seed=3)
        dt = torch.float32 if prec == "mixed" else torch.float64
        for x, r in zip(gt.vjp(*[_t(v, dt) for v in g]), ot.vjp(*g)):
            assert np.abs(_np(x).astype(np.float64) - r).max() <= VTOL[prec] * max(np.abs(r).max(), 1e-300)
    gt.destroy()


@pytest.mark.parametrize("c", [2, 7, 8, 9, 11, 13, 16, 17, 25, 32, 33, 49, 57, 64, 65, 130])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("det", [False, True])
def test_vjp_by_leaf_size(c, prec, det):
    """Leaves at the limits of the one, two, four and eight segments that the
    VJP's rows take, and of one pass of sinks: four mirrored quarters, every leaf with
    exactly c particles, some of them in reach of the others' support."""
    import torch
    from paper_1108_0028_amd import Tree
    _say("leaf size", c, prec, det)
    q = W.small_random(c, 70 + c, "uniform", h_scale=4.0)
    x, y = 2.0 + np.abs(q.x), 1.0 + np.abs(q.y)
    X = np.concatenate([x, -x, x, -x])
    Y = np.concatenate([y, y, -y, -y])
    Z, m, h = (np.tile(v, 4) for v in (q.z, q.m, q.h))
    ot = O.OracleTree(X, Y, Z, m, h, n_ll=c)
    cnt = ot.topology()["count"]
    assert ot.n_leaves == 4 and (cnt[4:8] == c).all()
    ot.walk(0.0)
    g = W.cotangents(4 * c, seed=5)
    dt = torch.float32 if prec == "mixed" else torch.float64
    gt = Tree(*[_t(v) for v in (X, Y, Z, m, h)], n_ll=c, theta=0.0, precision=prec, deterministic=det)
    for a, r in zip(gt.vjp(*[_t(v, dt) for v in g]), ot.vjp(*g)):
        assert np.abs(_np(a).astype(np.float64) - r).max() <= VTOL[prec] * np.abs(r).max()
    gt.destroy()
