"""Sorting of neighbour lists of more than 256 ids: by a bitmap of the caller's
indices for clouds of up to 262,144 particles, by a network above. 700 particles
with wide supports at scattered caller indices, among many with no neighbours;
the CSR must equal the all-pairs search exactly. (Lists past the 4096 ids that
threads keep, and lists searched again, are in the overflow test.)"""
import numpy as np
import pytest

import workloads as W

from test_gpu_parity import _gpu_tree, _np, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [701, 262144, 262145])
def test_long_lists_by_cloud_size(n):
    _say("long lists", n)
    rng = np.random.default_rng(n)
    p = rng.uniform(-1, 1, (n, 3))
    h = np.full(n, 1e-7)
    hot = np.sort(rng.choice(n, 700, replace=False))
    hot[0], hot[-1] = 0, n - 1   # the first and the last bit
    p[hot] = 0.002 * rng.normal(size=(700, 3))
    h[hot] = rng.uniform(0.002, 0.02, 700)
    x, y, z = (np.ascontiguousarray(v) for v in p.T)
    gt = _gpu_tree(W.Cloud("hot", x, y, z, np.full(n, 1.0 / n), h), 12, 0.7)
    off, ids = (_np(v) for v in gt.neighbours())
    cnt = np.diff(off)
    want = np.zeros(n, np.int64)
    for a in hot:
        r2 = ((x - x[a]) * (x - x[a]) + (y - y[a]) * (y - y[a])) + (z - z[a]) * (z - z[a])
        near = np.flatnonzero(r2 < (2.0 * h[a]) * (2.0 * h[a]))
        near = near[near != a]
        want[a] = len(near)
        np.testing.assert_array_equal(ids[off[a]:off[a + 1]], near)
    np.testing.assert_array_equal(cnt, want)
    assert (want > 256).sum() > 300
    gt.destroy()


@pytest.mark.parametrize("nll", [5, 10, 20, 50])
def test_lists_by_waves_per_leaf(nll):
    """8192, 4096 and 2048 leaves take one, two and four waves each; leaves of
    more than 32 particles take their sinks in several passes."""
    from oracle import oracle as O
    _say("waves per leaf", nll)
    c = W.clumpy_cube(40000)
    ot = O.OracleTree(*c.arrays(), n_ll=nll)
    ot.walk(0.7)
    ooff, oids, valid = ot.neighbours()
    assert valid.all() and np.diff(ooff).max() > 256
    gt = _gpu_tree(c, nll, 0.7)
    off, ids = gt.neighbours()
    np.testing.assert_array_equal(_np(off), ooff)
    np.testing.assert_array_equal(_np(ids), oids)
    gt.destroy()
