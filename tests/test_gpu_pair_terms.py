"""Deterministic VJP: the two sides of a near pair, which two kernels form, are
the same bits. Two particles and theta = 0: dx_0 = K_10 - K_01 and dx_1 = K_01 -
K_10 in FP64 sums of one rounded K each, so they are opposite exactly."""
import numpy as np
import pytest

from test_gpu_parity import _say
from test_gpu_vjp import _np, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nll", [1, 2])
def test_sides_of_a_pair_are_opposite(prec, nll):
    import torch
    from paper_1108_0028_amd import Tree
    _say("sides of a pair", prec, nll)
    rng = np.random.default_rng(3)
    dt = torch.float32 if prec == "mixed" else torch.float64
    for i in range(120):
        # within the support (both pieces of the spline), at its edge and outside
        r = rng.normal(size=(2, 3)) * 10.0 ** rng.uniform(-1.0, 0.5)
        a = [r[:, 0], r[:, 1], r[:, 2], rng.uniform(0.1, 2.0, 2), rng.uniform(0.3, 1.5, 2)]
        t = Tree(*[_t(v) for v in a], n_ll=nll, theta=0.0, precision=prec, deterministic=True)
        dx, dy, dz, _ = t.vjp(*[_t(rng.normal(size=2), dt) for _ in range(3)])
        for d in (dx, dy, dz):
            d = _np(d)
            assert d[0] != 0.0 and d[0] == -d[1], (i, d)
        t.destroy()
