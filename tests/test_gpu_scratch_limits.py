"""Calls whose scratch the caller's allocator refuses in its first size: gravity
takes ranges of groups with a smaller buffer for their far coefficients, refresh
gathers from the input arrays instead of from records of them. Results as
without a limit, bit for bit."""
import ctypes as C

import numpy as np
import pytest

import workloads as W

from test_gpu_parity import _say
from test_zz_no_alloc import _Counting, _build, _export

pytestmark = pytest.mark.gpu


class _Limited(_Counting):
    def __init__(self):
        super().__init__()
        import torch
        from paper_1108_0028_amd import _lib
        self.limit = 1 << 62
        self.refused = 0

        def alloc(nbytes, stream, ctx):
            if nbytes > self.limit:
                self.refused += 1
                return None
            return torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(), stream or 0)

        self.alloc_fn = _lib._ALLOC_FN(alloc)


@pytest.mark.parametrize("n,nll", [(9000, 8), (700, 90)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("limit", [300, 3000, 20000])
def test_gravity_and_refresh(n, nll, prec, limit):
    import torch
    from paper_1108_0028_amd import Tree
    from paper_1108_0028_amd._lib import _check, _ptr, _stream, lib
    _say("scratch limits", n, nll, prec, limit)
    L = lib()
    dev = torch.device("cuda:0")
    dt = torch.float32 if prec == "mixed" else torch.float64
    c = W.small_random(n, 17, "clustered")
    arrs = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in c.arrays()]
    ref = Tree(*arrs, n_ll=nll, theta=0.6, precision=prec)
    lim = _Limited()
    h = _build(arrs, nll, 0.6, prec, lim)
    _check(L.rcb_walk(h, _stream()), "rcb_walk")
    want = ref.gravity()
    acc = [torch.empty(n, dtype=dt, device=dev) for _ in range(3)]
    lim.limit = limit
    st = L.rcb_gravity(h, *[_ptr(a) for a in acc], _stream())
    torch.cuda.synchronize()
    leaves = 1 << ref.info()["k"]
    group = 22 * 8 * min(8, leaves)   # one group's coefficients
    if limit < group:
        assert st != 0
    else:
        assert st == 0 and (lim.refused > 0 or limit >= 22 * 8 * leaves)
        for a, b in zip(acc, want):
            np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    # a refresh whose records are refused
    moved = [a * 1.0001 for a in arrs]
    ref.refresh(*moved)
    need = L.rcb_refresh_noalloc_scratch(h)
    lim.limit, lim.refused = need + 16 * n, 0
    _check(L.rcb_refresh(h, *[_ptr(a) for a in moved], n, 0, _stream()), "rcb_refresh")
    assert lim.refused == 1
    lim.limit = 1 << 62
    nlab = ref.info()["n_labels"]
    for f in ("com", "mass", "quad"):
        w = ref.export(f)
        got = _export(h, f, w).reshape(nlab, -1)[1:]
        np.testing.assert_array_equal(got, w.cpu().numpy().reshape(nlab, -1)[1:])
    L.rcb_destroy(h, _stream())
    ref.destroy()
