"""Mixed form: the sum of a deep node's adjoint, added in FP64. One light particle
far out on the diagonal of a cube of 2^17 - 1 others (N_ll = 1, k = 17) ends in a leaf
whose box shrinks to a point, and no node above level 17 that holds it is small
enough for the MAC: all 16,384 groups add to the adjoint of that leaf, and the
particle's dm is their sum. What is asked for is that of eight FP32 parts of 2048
terms of one sign: each addition rounding by at most half an ulp of the part
(uniformly: 2^-23 / sqrt(12) of it, an ulp being 0.72 times that on average), a part is
off by 2^-23 0.72 / sqrt(12) sqrt(2048 / 3) = 6.5e-7 and their sum by 2.3e-7 (rms); in
one part of 16,384 it would be 1.8e-6. The bar, 6e-7 rms over twelve cotangents, lies
a factor of three from either."""
import numpy as np
import pytest

import workloads as W

from test_gpu_parity import _say
from test_gpu_vjp import _np, _t

pytestmark = pytest.mark.gpu


def _cloud(n=1 << 17):
    rng = np.random.default_rng(1)
    p = rng.uniform(0.0, 1.0, (n, 3))
    p[-1] = 8.0
    m = np.full(n, 1.0 / n)
    m[-1] *= 0.05
    return W.Cloud("outlier", *[np.ascontiguousarray(p[:, i]) for i in range(3)], m,
                   np.full(n, 0.2 * n ** (-1.0 / 3.0)))


def test_deep_node_adjoint():
    import torch
    from paper_1108_0028_amd import Tree
    c = _cloud()
    _say("deep node adjoint", c.n)
    arrs = [_t(a) for a in c.arrays()]
    exact = Tree(*arrs, n_ll=1, theta=0.5)
    mixed = Tree(*arrs, n_ll=1, theta=0.5, precision="mixed")
    # the leaf of the last particle is in (nearly) every leaf's far list, no
    # ancestor of it is
    nl = 1 << exact.info()["k"]
    assert nl == 1 << 17
    pos = int((exact.export("perm") == c.n - 1).nonzero()[0])
    first, count = exact.export("first")[nl:], exact.export("count")[nl:]
    leaf = nl + int(((first <= pos) & (pos < first + count)).nonzero()[0])
    far = exact.export("far")
    live = int((count > 0).sum())
    assert int((far == leaf).sum()) > 0.99 * live
    assert all(int((far == (leaf >> u)).sum()) == 0 for u in range(1, 18))
    rng = np.random.default_rng(2)
    err = []
    for _ in range(12):
        d = np.ones(3) / np.sqrt(3.0) + 0.3 * rng.normal(size=3)
        g = [_t((v + 0.1 * rng.normal(size=c.n)).astype(np.float32)) for v in d]
        ref = float(_np(exact.vjp(*[v.double() for v in g])[3])[-1])
        err.append(float(_np(mixed.vjp(*g)[3])[-1]) / ref - 1.0)
    rms = float(np.sqrt(np.mean(np.square(err))))
    print(f"   dm of the outlier: rms error {rms:.2e}", flush=True)
    assert rms <= 6e-7
    exact.destroy()
    mixed.destroy()
