"""The subtrees of the device build at the edges of what one workgroup holds:
2048 particles and 8 levels by eight waves for clouds of at most 2^18
particles, 1024 and 7 by four above. Chunks of a wave (512 particles) and
their combination, leaves of more than one chunk, roots just above the limit,
empty subtrees and more levels than one workgroup takes; the tree and its
lists as the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from test_gpu_parity import _gpu_tree, _say, compare_lists, compare_trees

pytestmark = pytest.mark.gpu

SIZES = [(1, 8), (9, 1), (511, 8), (512, 8), (513, 8), (1025, 600), (1500, 1500), (1537, 8), (2047, 1), (2048, 8),
         (2048, 2048), (2049, 8), (2049, 1025), (5000, 1200), (4097, 1)]


@pytest.mark.parametrize("n,nll", SIZES)
@pytest.mark.parametrize("kind", ["uniform", "clustered"])
def test_subtree_edges(n, nll, kind):
    _say("subtree", n, nll, kind)
    c = W.small_random(n, 900 + n, kind)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.7)
    gt = _gpu_tree(c, nll, 0.7)
    compare_trees(gt, ot)
    compare_lists(gt, ot)
    gt.destroy()


@pytest.mark.parametrize("n,nll", [(2000, 2), (6000, 3)])
def test_subtree_coincident(n, nll):
    """Particles at three points only: one child takes everything, level after
    level, and the other one's subtree is empty."""
    _say("coincident", n, nll)
    c = W.small_random(n, 31, "uniform")
    x, y, z, m, h = (np.array(v) for v in c.arrays())
    for a in (x, y, z):
        a[:] = a[np.arange(n) % 3]
    c = W.Cloud("coincident", x, y, z, m, h)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    gt = _gpu_tree(c, nll, 0.7)
    compare_trees(gt, ot)
    gt.destroy()


@pytest.mark.parametrize("n,nll", [(1 << 18, 700), ((1 << 18) + 1, 9), ((1 << 18) + 1, 700)])
def test_subtree_rule(n, nll):
    _say("rule", n, nll)
    c = W.small_random(n, 7, "uniform")
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    gt = _gpu_tree(c, nll, 0.7)
    compare_trees(gt, ot)
    gt.destroy()


@pytest.mark.parametrize("n,nll,sigma", [(2040, 8, 0.3), (2040, 8, 0.6), (2040, 8, 1.0), (2040, 8, 2.0), (5000, 6, 0.6)])
def test_subtree_uneven(n, nll, sigma):
    """Coordinates with a long tail: the nodes of a level hold from none to
    hundreds of particles, and take lanes each to its size."""
    _say("uneven", n, nll, sigma)
    rng = np.random.default_rng(int(100 * sigma) + n)
    x, y, z = np.exp(sigma * rng.normal(size=(3, n)))
    c = W.Cloud("uneven", x, y, z, rng.uniform(0.5, 1.5, n) / n, rng.uniform(0.05, 0.15, n))
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.7)
    for prec in ("fp64", "mixed"):
        gt = _gpu_tree(c, nll, 0.7, prec)
        compare_trees(gt, ot)
        compare_lists(gt, ot)
        gt.destroy()
