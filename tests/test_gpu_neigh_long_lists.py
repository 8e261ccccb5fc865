"""Lists of more than 4096 ids in a cloud past the sizes whose lists a bitmap sorts
(2^18 particles): 5000 particles in a clump that each one's support spans. Sorted in
place in the CSR by one workgroup each, after the copy from the pool's chains, and, in
the smallest scratch, where the pool runs out, after a search of their own. The CSR is
the oracle's."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import _np, _say
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu

N, CLUMP = (1 << 18) + 517, 5000


def _cloud():
    rng = np.random.default_rng(8)
    p = rng.uniform(-1.0, 1.0, (N, 3))
    h = np.full(N, 0.5 * (20.0 * 8.0 / (4.19 * N)) ** (1 / 3))
    who = rng.permutation(N)[:CLUMP]
    p[who] = 0.3 + 1e-3 * rng.uniform(-1.0, 1.0, (CLUMP, 3))
    h[who] = 2e-3
    return W.Cloud("clump", *[np.ascontiguousarray(p[:, i]) for i in range(3)], np.full(N, 1.0 / N), h)


@pytest.mark.parametrize("smallest", [False, True])
def test_long_lists(smallest, monkeypatch):
    _say("long lists of a large cloud", smallest)
    c = _cloud()
    ot = O.OracleTree(*c.arrays(), n_ll=12)
    ot.walk(0.7)
    off, ids, valid = ot.neighbours()
    assert valid.all() and int((np.diff(off) > 4096).sum()) >= CLUMP
    lim = LimitedAlloc()
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=12, theta=0.7)
    t.walk()
    o = _t(np.full(N + 1, -1, np.int64))
    if smallest:   # rows, heads, N / 8 chunks, queue and the scan of the counts
        lim.budget = lim.live + 260 * N + 272 * (N // 8 + 1) + 4 * (1 << t.info()["k"]) + 8 * (N // 2048 + 1) + 256
    total = t.neighbours_count(o)
    assert total == len(ids) and (lim.refused > 0) == smallest
    lim.budget = 1 << 62
    i = _t(np.full(total, -1, np.int32))
    for _ in range(2):
        t.neighbours_fill(o, i)
        np.testing.assert_array_equal(_np(o), off)
        np.testing.assert_array_equal(_np(i), ids)
    t.destroy()
