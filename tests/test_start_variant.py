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
F64, F32, BF16 = dict(wdtype=0, fdtype=0), dict(wdtype=1, fdtype=1), dict(wdtype=1, fdtype=2)


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


@pytest.mark.parametrize("N,kw,lds", [
    (80000, dict(n=25), SMALL), (80001, dict(n=25), STAGED), (80000, dict(n=25, mode=2), SMALL),
    (62500, dict(n=25, m=4, hv_alpha=3), SMALL), (70225, dict(n=25, m=4, hv_alpha=3), STAGED),
    (42000, dict(n=120), SMALL), (52900, dict(n=60), STAGED),
    (46656, dict(dim=3, n=20, hv_alpha=1), SMALL), (54872, dict(dim=3, n=20, hv_alpha=1), STAGED),
    (35937, dict(dim=3, n=35), SMALL), (46656, dict(dim=3, n=35), STAGED),
    (27000, dict(dim=3, n=110), SMALL), (35937, dict(dim=3, n=60), STAGED)])
def test_fp64(N, kw, lds):
    assert _variant(N, **F64, **kw) == (lds, 256)
