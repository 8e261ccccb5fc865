"""Prefix sums of the neighbour counts by one workgroup (up to 16,384 particles) and
by blocks: the offsets are the sums of the lists' lengths."""
import numpy as np
import pytest

import workloads as W

from test_gpu_parity import _gpu_tree, _np, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 8191, 8193, 16384, 16385, 18433, 1 << 20])
def test_offsets(n):
    _say("scan", n)
    rng = np.random.default_rng(n)
    x, y, z = rng.uniform(-1, 1, (3, n))
    # pairs of neighbours at scattered caller indices: each of a pair lists the other
    pairs = rng.permutation(n)[:2 * (n // 3)].reshape(-1, 2) if n > 2 else np.empty((0, 2), int)
    for a in (x, y, z):
        a[pairs[:, 1]] = a[pairs[:, 0]] + 1e-9
    h = np.full(n, 1e-8)
    want = np.zeros(n, np.int64)
    want[pairs.ravel()] = 1
    other = np.full(n, -1)
    other[pairs[:, 0]], other[pairs[:, 1]] = pairs[:, 1], pairs[:, 0]
    gt = _gpu_tree(W.Cloud("pairs", x, y, z, np.full(n, 1.0 / n), h), 12, 0.9)
    off, ids = (_np(v) for v in gt.neighbours())
    np.testing.assert_array_equal(off, np.concatenate([[0], np.cumsum(want)]))
    np.testing.assert_array_equal(ids, other[want > 0])
    gt.destroy()
