"""Interaction lists longer than the walk's slabs: at theta = 0 every cell is
near to every group, so the near lists of this cloud (more than 16384 entries)
outgrow the slab, their groups outgrow both queues of the wide walk, and the
lists are walked a second time into exact storage. Forces and neighbour counts
equal the sum and the search over all pairs."""
import numpy as np
import pytest

import workloads as W

from test_gpu_parity import _say
from test_gpu_vjp import _t

pytestmark = pytest.mark.gpu


def _pair_sums(x, m, h, rows):
    """accelerations and neighbour counts of all particles by plain FP64 torch"""
    import torch
    acc, cnt = torch.empty_like(x), torch.empty(x.shape[0], dtype=torch.int64, device=x.device)
    for s in range(0, x.shape[0], rows):
        v = x[s:s + rows, None, :] - x[None, :, :]
        r2 = (v[..., 0] * v[..., 0] + v[..., 1] * v[..., 1]) + v[..., 2] * v[..., 2]
        own = 2.0 * h[s:s + rows, None]
        cnt[s:s + rows] = (r2 < own * own).sum(1) - 1
        hi = 2.0 / (h[s:s + rows, None] + h[None, :])
        r = torch.sqrt(r2)
        q = r * hi
        near = hi ** 3 * (4 / 3 - 1.2 * q ** 2 + 0.5 * q ** 3)
        mid = hi ** 3 * (8 / 3 - 3 * q + 1.2 * q ** 2 - q ** 3 / 6) - r ** -3 / 15
        f = torch.where(q < 1, near, torch.where(q < 2, mid, r ** -3))
        acc[s:s + rows] = -((m * f)[..., None] * v).sum(1)
    return acc, cnt


def test_lists_past_the_slabs():
    import torch
    from paper_1108_0028_amd import Tree
    c = W.small_random(36000, 17, "uniform", h_scale=0.2)
    arrs = [_t(v) for v in c.arrays()]
    _say("walk: exact lists", c.n)
    t = Tree(*arrs, n_ll=1, theta=0.0)
    assert int((t.export("count")[1 << t.info()["k"]:] > 0).sum()) > 16384
    off, ids = t.neighbours()
    acc = torch.stack(t.gravity(), 1)
    ref, cnt = _pair_sums(torch.stack(arrs[:3], 1), arrs[3], arrs[4], 500)
    assert torch.equal(off[1:] - off[:-1], cnt)
    assert t.info()["walk_requeued"] > 0
    # 36000 terms a sum: n u = 8e-12 of the terms' sum, which the cloud's balance
    # makes some tens of times its result; rms over the particles
    assert float((acc - ref).norm() / ref.norm()) < 1e-11
    t.destroy()
