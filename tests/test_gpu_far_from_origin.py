"""A cloud so far from the origin that the square of its distance is past the
range of FP64: moments are taken about each node's centre of mass, so the tree is
the oracle's all the same, bit for bit -- built by subtrees and level by level,
and refreshed; cells of one chunk of 512 particles, of less and of more."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from test_gpu_parity import _gpu_tree, _say, compare_trees
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


def _far(c):
    s = lambda v: 1e155 + 1e147 * v
    return W.Cloud("far", s(c.x), s(c.y), s(c.z), c.m, 1e147 * c.h)


@pytest.mark.parametrize("levels", [False, True])
@pytest.mark.parametrize("n,nll", [(1, 12), (700, 12), (3000, 900), (5000, 6), (20000, 40)])
def test_tree(n, nll, levels, monkeypatch):
    if levels:
        monkeypatch.setenv("RCB_BUILD_LEVELS", "1")
    _say("far from the origin", n, nll, levels)
    c = _far(W.small_random(n, 31 + n, "clustered"))
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    assert np.isfinite(ot.nodes()["Q"][1:]).all()
    gt = _gpu_tree(c, nll, 0.7)
    compare_trees(gt, ot)
    gt.refresh(*[_t(a) for a in c.arrays()])
    compare_trees(gt, ot)
    gt.destroy()
