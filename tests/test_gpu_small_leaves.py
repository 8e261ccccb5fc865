"""Leaves of one or two particles, whose near field takes its sources lane by lane,
next to leaves of more in the same tree; groups of waves from one to eight. Against
the oracle, and the sum over all pairs at theta = 0, coincident particles included."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from test_gpu_parity import TOL, _gpu_tree, _np, _say, gate

pytestmark = pytest.mark.gpu


# cells: 1 to 32,768; the wave counts change at 1024 cells, and with five and two
# and a half particles a cell (theta = 0, the sum over all pairs, for the smaller clouds)
SMALL = [(1, 1), (2, 1), (2, 2), (3, 2), (65, 1), (700, 1), (1500, 2), (2600, 2)]
CASES = [(n, nll, th) for n, nll in SMALL for th in (0.0, 0.6)] + [(9000, 5, 0.6), (11000, 5, 0.6), (20000, 1, 0.6)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,nll,theta", CASES)
def test_small_leaves(n, nll, theta, prec):
    c = W.small_random(n, 300 + n, "uniform" if n % 2 else "clustered", h_scale=0.5)
    if n > 60:
        for a in (c.x, c.y, c.z):
            a[20:22] = a[19]
    _say("small leaves", n, nll, theta, prec)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(theta)
    ref = np.stack(ot.gravity(), 1)
    gt = _gpu_tree(c, nll, theta, prec)
    assert gate(np.stack([_np(a) for a in gt.gravity()], 1), ref) <= TOL[prec]
    gt.destroy()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("same", [64, 65, 1500])
def test_a_large_leaf_among_them(same, prec):
    """(2048 cells: the rule for small leaves ends at 64 particles in one)"""
    c = W.small_random(4000, 305, "uniform", h_scale=0.5)
    for a in (c.x, c.y, c.z):
        a[100:100 + same] = a[99]
    _say("a large leaf among small ones", same, prec)
    ot = O.OracleTree(*c.arrays(), n_ll=2)
    ot.walk(0.6)
    ref = np.stack(ot.gravity(), 1)
    gt = _gpu_tree(c, 2, 0.6, prec)
    assert int(gt.export("count")[1 << ot.k:].max()) > same
    assert gate(np.stack([_np(a) for a in gt.gravity()], 1), ref) <= TOL[prec]
    gt.destroy()
