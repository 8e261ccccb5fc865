"""Reading B has no VJP, so its gravity call keeps nothing: the tree holds as much
workspace after it as before, and repeats the forces bit for bit."""
import pytest

import workloads as W

from limited_alloc import LimitedAlloc
from test_gpu_parity import _say
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reading", ["A", "B"])
def test_gravity_keeps_coefficients_for_a_vjp_only(reading, monkeypatch):
    import torch
    _say("workspace after gravity, reading", reading)
    lim = LimitedAlloc()
    c = W.small_random(5000, 71, "clustered")
    t = lim.tree(monkeypatch, [_t(a) for a in c.arrays()], n_ll=8, theta=0.6, taylor_reading=reading)
    t.walk()
    held = lim.live
    acc = t.gravity()
    assert lim.live - held == (22 * 8 * (1 << t.info()["k"]) if reading == "A" else 0)
    for a, b in zip(acc, t.gravity()):
        assert torch.equal(a, b)
    t.destroy()
