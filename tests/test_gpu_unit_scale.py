"""The FP64 form has no length scale of its own: with positions and smoothing
lengths times a power of two every rounding stays as it was, so accelerations
(s^-2) and gradients (s^-3; of the masses s^-2) are the unscaled ones times
that power, bit for bit, however small or large the units are -- coincident
particles, and particles farther than their support from their cell's centre,
included."""
import numpy as np
import pytest

import workloads as W

from test_gpu_parity import _say
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


def _cloud(scale, h_scale):
    c = W.small_random(1500, 23, "clustered", h_scale=h_scale)
    for a in (c.x, c.y, c.z):
        a[10:13] = a[9]          # coincident particles
    return [_t(a * scale) for a in (c.x, c.y, c.z)] + [_t(c.m), _t(c.h * scale)]


@pytest.mark.parametrize("log2s", [-77, -73, 70])      # 6.6e-24, 1.1e-22, 1.2e21
@pytest.mark.parametrize("nll,h_scale", [(8, 1.0), (8, 0.05), (60, 0.3)])
def test_gravity(log2s, nll, h_scale):
    import torch
    from paper_1108_0028_amd import Tree
    _say("gravity in units of 2 **", log2s, nll, h_scale)
    s = 2.0 ** log2s
    for theta in (0.0, 0.6):
        one = Tree(*_cloud(1.0, h_scale), n_ll=nll, theta=theta)
        t = Tree(*_cloud(s, h_scale), n_ll=nll, theta=theta)
        for a, b in zip(t.gravity(), one.gravity()):
            assert bool(torch.isfinite(b).all())
            assert torch.equal(a * s * s, b)
        t.destroy()
        one.destroy()


# theta = 0: the far field's adjoint holds r^-13, past the range of FP64 in
# such units
@pytest.mark.parametrize("log2s", [-77, -73, 70])
@pytest.mark.parametrize("nll,h_scale", [(8, 1.0), (8, 0.05), (60, 0.3)])
@pytest.mark.parametrize("det", [False, True])
def test_vjp(log2s, nll, h_scale, det):
    import torch
    from paper_1108_0028_amd import Tree
    _say("gradients in units of 2 **", log2s, nll, h_scale, det)
    s = 2.0 ** log2s
    g = [_t(v) for v in W.cotangents(1500, seed=5)]
    one = Tree(*_cloud(1.0, h_scale), n_ll=nll, theta=0.0, deterministic=det)
    t = Tree(*_cloud(s, h_scale), n_ll=nll, theta=0.0, deterministic=det)
    for a, b, f in zip(t.vjp(*g), one.vjp(*g), (s ** 3, s ** 3, s ** 3, s ** 2)):
        assert bool(torch.isfinite(b).all())
        if det:
            assert torch.equal(a * f, b)
        else:    # 1500 terms added in any order: n u of the largest, and a margin of 10
            assert float((a * f - b).abs().max()) <= 1500 * 10 * 2.0 ** -53 * float(b.abs().max())
    t.destroy()
    one.destroy()
