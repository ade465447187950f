"""Runs whose steps are one kernel each (staged 2D FP32 plans) against the
global-gather kernels, bit for bit, with everything a run folds in: one tile, a
few, one round of workgroups and several; few and many weights, halos that wrap;
and two runs at once on one workspace, whose flags overwrite each other so that
workgroups compute what they miss."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


def _solver(shape, n, m, alpha, bc):
    xyz, flags, h = nodes.jittered_grid(shape, seed=3, periodic=bc == "PERIODIC")
    return Solver(2, xyz, flags, h, n, m, alpha, 1e-4 / (configs.SC * h), (0.0,) * 2, (1.0,) * 2, precision="f32", bc=bc)


@pytest.mark.parametrize("shape,n,m,alpha,bc", [
    ((9, 8), 12, 2, 2, "PEC"), ((16, 16), 25, 2, 2, "PEC"), ((50, 41), 25, 4, 3, "PERIODIC"), ((211, 190), 31, 4, 2, "PEC"),
    ((367, 363), 25, 2, 2, "PERIODIC"), ((600, 607), 13, 2, 2, "PEC"), ((600, 607), 25, 4, 3, "PERIODIC"),
    ((1003, 997), 25, 2, 2, "PEC")])
def test_whole_steps_equal_halves(shape, n, m, alpha, bc):
    s = _solver(shape, n, m, alpha, bc)
    rs = np.random.RandomState(n)
    E0, H0 = rs.standard_normal(s.N), rs.standard_normal((s.N, 2))
    T = 7
    src = (rs.randint(0, s.N, 3), np.array([1.0, -0.5, 2.0]), rs.standard_normal((T, 3)))
    rcv = rs.randint(0, s.N, 70)
    eps = 1 + rs.uniform(size=s.N) if n % 2 else None
    out = []
    for lds in (0, 1):
        s.set_variant(block=256, xcd=1, lds=lds)
        st = s.state(E0, H0, eps_r=eps)
        r = s.run(st, T, src=src, rcv=rcv, energy_every=3)
        s.run(st, 4)
        out.append((st.E.clone(), st.H.clone(), r["traces"], r["energy"]))
    for a, b in zip(out[1][:3], out[0][:3]):
        assert torch.equal(a, b)
    assert np.array_equal(out[1][3], out[0][3])


def test_two_runs_at_once():
    s = _solver((367, 363), 25, 2, 2, "PEC")
    rs = np.random.RandomState(1)
    fields = [(rs.standard_normal(s.N), rs.standard_normal((s.N, 2))) for _ in range(2)]
    s.set_variant(block=256, xcd=1, lds=0)
    ref = [s.state(*f) for f in fields]
    for st in ref:
        s.run(st, 40)
    s.set_variant(block=256, xcd=1, lds=1)
    got = [s.state(*f) for f in fields]
    streams = [torch.cuda.Stream() for _ in got]
    torch.cuda.synchronize()
    for q, st in zip(streams, got):
        with torch.cuda.stream(q):
            s.run(st, 40)
    torch.cuda.synchronize()
    for a, b in zip(got, ref):
        assert torch.equal(a.E, b.E) and torch.equal(a.H, b.H)
