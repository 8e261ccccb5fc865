"""Host build of the workgroup renumbering (csrc/xcd_map.h): every launch size
is taken once and only once, one XCD's workgroups are contiguous ranges or runs,
around the size from which runs are taken and with every kind of remainder."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SHIM = os.path.join(HERE, "native", "xcd_map_shim.cpp")
OUT = os.path.join(HERE, "native", "_build", "libxcd_map_shim.so")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1108_0028_amd", "csrc")


def _slots(nb, run):
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    srcs = [SHIM, os.path.join(CSRC, "xcd_map.h")]
    if not os.path.exists(OUT) or os.path.getmtime(OUT) < max(map(os.path.getmtime, srcs)):
        subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-std=c++17", "-I", CSRC, "-o", OUT, SHIM])
    L = C.CDLL(OUT)
    out = np.empty(nb, np.uint32)
    L.shim_xcd_slots(C.c_uint32(nb), C.c_uint32(run), out.ctypes.data_as(C.c_void_p))
    return out


@pytest.mark.parametrize("run", [1, 8, 64])
@pytest.mark.parametrize("rounds", [0, 1, 511, 512, 513, 8192])
@pytest.mark.parametrize("rest", [-9, -1, 0, 1, 7, 8, 63, 65, 509])
def test_every_workgroup_once(run, rounds, rest):
    nb = 8 * run * rounds + rest
    if nb < 1:
        nb = 8 * run * rounds + 10 + rest
    s = _slots(nb, run)
    assert np.array_equal(np.sort(s), np.arange(nb, dtype=np.uint32))
    for x in range(8):   # breaks in an XCD's sequence: none, or between runs
        brk = np.flatnonzero(np.diff(s[x::8].astype(np.int64)) != 1) + 1
        assert np.all(brk % run == 0)
        assert nb >= 4096 * run or len(brk) == 0
