"""3D small-set kernels (lds = 3) against the staged (1, 2) and global (0) ones:
FP32 and BF16 bit for bit (one order of summation), FP64 to the rounding of
another order; node counts around the 64-node tile, chunk counts below, at
and above the nine a wavefront holds and the sixteen two rounds fetch, curl
stencils longer and shorter than the hyperviscosity's, no hyperviscosity."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


def _run(s, E0, H0, lds, T, src, rcv):
    s.set_variant(block=256, xcd=1, lds=lds)
    st = s.state(E0, H0)
    out = s.run(st, T, src=src, rcv=rcv)
    return st.E.clone(), st.H.clone(), out["traces"]


@pytest.mark.parametrize("shape,n,alpha,n_hv", [
    ((5, 5, 5), 35, 2, 71), ((6, 6, 7), 26, 1, 27), ((8, 9, 7), 35, 1, 27), ((7, 8, 9), 65, 1, 41),
    ((7, 9, 11), 35, 2, 71), ((9, 9, 5), 35, 2, 90), ((6, 7, 8), 30, 0, 0)])
@pytest.mark.parametrize("precision", ["f64", "f32", "bf16"])
def test_small_set_3d(shape, n, alpha, n_hv, precision):
    rs = np.random.RandomState(n)
    xyz, flags, h = nodes.jittered_grid(shape, seed=5)
    s = Solver(3, xyz, flags, h, n, 2, alpha, 1e-3 / (configs.SC * h), (0.0,) * 3, (1.0,) * 3, n_hv=n_hv,
               precision=precision)
    E0, H0 = rs.standard_normal((s.N, 3)), rs.standard_normal((s.N, 3))
    T = 3
    src = (rs.randint(0, s.N, 2), np.array([1.0, -0.5]), rs.standard_normal((T, 2)))
    rcv = rs.randint(0, s.N, 70)
    ref = _run(s, E0, H0, 1, T, src, rcv)
    small = _run(s, E0, H0, 3, T, src, rcv)
    for a, b in zip(small, ref):
        if precision == "f64":
            # three steps of sums of at most ~360 products, each within a few ulp of the other's
            assert float((a - b).abs().max()) <= 1e-12 * float(b.abs().max())
        else:
            assert torch.equal(a, b)
