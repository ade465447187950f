"""Staged kernels whose operator stays in cache (ordinary loads), lies in the
band that streams all the same, or exceeds the memory-side cache, with the E
update over the tiles in reverse: bit for bit the global-gather kernels, which
go forward; tile counts off every multiple of 8, with and without the remap."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


# 2D FP32: streaming below 120k nodes, in the band and above the cache, cached between; FP64 and 3D cached
@pytest.mark.parametrize("shape,n,precision", [
    ((9, 8), 12, "f32"), ((50, 41), 25, "f64"), ((211, 190), 25, "f32"), ((367, 363), 25, "f32"), ((367, 363), 60, "f32"),
    ((884, 871), 25, "f32"), ((211, 190), 12, "f64"), ((13, 12, 11), 35, "f32"), ((17, 15, 11), 35, "f64")])
@pytest.mark.parametrize("xcd", [0, 1])
def test_staged_equals_global(shape, n, precision, xcd):
    dim = len(shape)
    xyz, flags, h = nodes.jittered_grid(shape, seed=3)
    s = Solver(dim, xyz, flags, h, n, 2, 2, 1e-4 / (configs.SC * h), (0.0,) * dim, (1.0,) * dim, precision=precision)
    rs = np.random.RandomState(n)
    E0 = rs.standard_normal((s.N,) if dim == 2 else (s.N, 3))
    H0 = rs.standard_normal((s.N, dim))
    out = []
    for lds in (0, 1) if dim == 2 else (0, 1, 2):
        s.set_variant(block=256, xcd=xcd, lds=lds)
        st = s.state(E0, H0)
        s.step(st, 3)
        out.append((st.E.clone(), st.H.clone()))
    for E, H in out[1:]:
        assert torch.equal(E, out[0][0]) and torch.equal(H, out[0][1])
