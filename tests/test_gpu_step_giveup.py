"""Whole steps in which workgroups do not wait for their neighbours' H but compute it
themselves, bit for bit against the global-gather kernels: with no patience at all many
of them come to that, so the path is taken here and not only when streams happen to
meet.  The sets are those of test_gpu_whole_steps: each of them does take whole steps,
with and without tiles that come twice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import Solver  # noqa: E402
from paper_2508_18205_amd._abi import RbffdError  # noqa: E402
from synth import configs, nodes  # noqa: E402


def _solver(shape, n, m, alpha, bc):
    xyz, flags, h = nodes.jittered_grid(shape, seed=3, periodic=bc == "PERIODIC")
    return Solver(2, xyz, flags, h, n, m, alpha, 1e-4 / (configs.SC * h), (0.0,) * 2, (1.0,) * 2, precision="f32", bc=bc)


@pytest.mark.parametrize("shape,n,m,alpha,bc,twice", [
    ((9, 8), 12, 2, 2, "PEC", False), ((16, 16), 25, 2, 2, "PEC", False), ((50, 41), 25, 4, 3, "PERIODIC", False),
    ((211, 190), 31, 4, 2, "PEC", True), ((367, 363), 25, 2, 2, "PERIODIC", True), ((600, 607), 13, 2, 2, "PEC", True),
    ((600, 607), 25, 4, 3, "PERIODIC", True), ((1003, 997), 25, 2, 2, "PEC", True)])
def test_computed_by_the_waiting(shape, n, m, alpha, bc, twice):
    s = _solver(shape, n, m, alpha, bc)
    rs = np.random.RandomState(n)
    E0, H0 = rs.standard_normal(s.N), rs.standard_normal((s.N, 2))
    T = 7
    src = (rs.randint(0, s.N, 3), np.array([1.0, -0.5, 2.0]), rs.standard_normal((T, 3)))
    rcv = rs.randint(0, s.N, 70)
    eps = 1 + rs.uniform(size=s.N) if n % 2 else None
    out, late = [], []
    for lds, patience in ((0, 0), (1, 0), (1, 200)):
        s.set_variant(block=256, xcd=1, lds=lds)
        s.set_patience(patience)
        was = s.whole_steps()
        assert was["whole"] == (lds == 1)
        st = s.state(E0, H0, eps_r=eps)
        r = s.run(st, T, src=src, rcv=rcv, energy_every=3)
        out.append((st.E.clone(), st.H.clone(), r["traces"], r["energy"]))
        late.append(s.whole_steps()["late"] - was["late"])
    assert was["tiles"] == -(-s.N // 256) and (was["twice"] > 0) == twice
    # one round of a few hundred workgroups or more is never done in the order of dispatch
    assert late[0] == 0 and (late[1] > 0 or was["tiles"] < 100)
    for got in out[1:]:
        for a, b in zip(got[:3], out[0][:3]):
            assert torch.equal(a, b)
        assert np.array_equal(got[3], out[0][3])


def test_patience_is_checked():
    s = _solver((9, 8), 12, 2, 2, "PEC")
    with pytest.raises(RbffdError):
        s.set_patience(-1)
