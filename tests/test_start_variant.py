"""The launch variant a plan starts on, by size, precision and stencils (plans are made
on the host: no GPU).  Sizes beside each line where the measured order of two kernels
turns; tiny FP32 sets take one 64-node tile per workgroup, where four left most of the
chip idle (17.3 us per step at 1600 nodes, n = 60, against 14.3 staged and 14.2 so)."""
import ctypes as C
import os

import numpy as np
import pytest

from test_abi import _params

GLOBAL, STAGED, SMALL = 0, 1, 3
F32, BF16 = dict(wdtype=1, fdtype=1), dict(wdtype=1, fdtype=2)


def _variant(N, dim=2, **kw):
    from paper_2508_18205_amd import _abi
    if not os.path.exists(_abi.LIB_PATH):
        pytest.skip("librbffd.so not built")
    lib = _abi.load()
    p = _params(_abi, dim=dim, **kw)
    p.hi[2] = 1.0
    xyz = np.random.default_rng(0).uniform(size=(N, dim))
    flags = np.zeros(N, np.uint8)
    plan = C.c_void_p()
    h_set = (N, xyz.ctypes.data, flags.ctypes.data) if kw.get("mode") == 2 else (0, None, None)
    assert lib.rbffd_plan_create(C.byref(p), N, xyz.ctypes.data, flags.ctypes.data, *h_set, C.byref(plan)) == 0
    v = C.c_int32()
    assert lib.rbffd_get_variant(plan, C.byref(v)) == 0
    lib.rbffd_plan_destroy(plan)
    return (v.value >> 17) & 7, v.value & 0xFFFF


@pytest.mark.parametrize("N,kw,lds,block", [
    (256, dict(F32), GLOBAL, 64), (2601, dict(F32, n=60), GLOBAL, 64), (40000, dict(F32), GLOBAL, 64),
    (40001, dict(F32), GLOBAL, 256), (65536, dict(F32), GLOBAL, 256), (65537, dict(F32), STAGED, 256),
    (900, dict(BF16), GLOBAL, 64), (900, dict(wdtype=3, fdtype=1), GLOBAL, 64), (900, dict(F32, pol=1), GLOBAL, 64),
    (900, dict(F32, mode=2), GLOBAL, 256), (24576, dict(F32, dim=3, n=35), SMALL, 256),
    (24577, dict(F32, dim=3, n=35), GLOBAL, 64), (65537, dict(F32, dim=3, n=35), STAGED, 256)])
def test_fp32(N, kw, lds, block):
    assert _variant(N, **kw) == (lds, block)
