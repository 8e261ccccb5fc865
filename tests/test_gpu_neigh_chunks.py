"""Neighbour lists past the 64-slot row (Sec. 2.3.2 "Neighbour list"): kept in
chains of 64-slot chunks from sub-pools, sorted by one wave (up to 256 ids) or
one workgroup. The CSR must equal the all-pairs search exactly.

  sphere:  ~105 neighbours (the paper's Table 1): nearly every list takes a chunk
  chains:  ~330 neighbours, cells of more than 64 particles: chains of several
           chunks, and the sinks left over from a cell's first 64
  halo:    a tight core inside a sparse halo whose supports reach the core: the
           pool, sized from each cell's own density, runs out, so kept lists and
           lists searched again meet in one call
"""
import numpy as np
import pytest

from oracle import brute
import workloads as W

from test_gpu_parity import _gpu_tree, _np, _say

pytestmark = pytest.mark.gpu


def _cloud(kind):
    if kind == "sphere":
        return W.sobol_sphere(5000, n_neigh=105), 12
    if kind == "chains":
        return W.sobol_sphere(4000, n_neigh=400), 100
    rng = np.random.default_rng(5)
    p = np.concatenate([0.01 * rng.normal(size=(3000, 3)), rng.uniform(-1, 1, (1500, 3))])
    h = np.concatenate([np.full(3000, 0.0015), np.full(1500, 0.8)])
    x, y, z = (np.ascontiguousarray(v) for v in p.T)
    return W.Cloud("halo", x, y, z, np.full(4500, 1.0 / 4500), h), 12


@pytest.mark.parametrize("kind", ["sphere", "chains", "halo"])
def test_lists_in_chunks(kind):
    c, nll = _cloud(kind)
    _say("neighbour chunks", kind)
    boff, bids = brute.neighbours(c.x, c.y, c.z, c.h)
    cnt = np.diff(boff)
    assert (cnt > 64).mean() > 0.2 and (kind == "sphere" or cnt.max() > 256)
    gt = _gpu_tree(c, nll, 0.7)
    for _ in range(2):   # the second call reuses the rows and the pool
        off, ids = gt.neighbours()
        np.testing.assert_array_equal(_np(off), boff)
        np.testing.assert_array_equal(_np(ids), bids)
    gt.destroy()
