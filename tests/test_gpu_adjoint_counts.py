"""The adjoint with more sources or receivers than its node loops look through (16 and
64) takes kernels of their own for them: the same gradients, bit for bit, as with the
few that matter, the others being silent sources and receivers without a residual."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import AdjointProblem, MaxwellFn, Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_many_equal_few(precision):
    xyz, flags, h = nodes.jittered_grid((23, 17), seed=3)
    s = Solver(2, xyz, flags, h, 12, 2, 2, 1e-3 / (configs.SC * h), (0.0,) * 2, (1.0,) * 2, precision=precision, adjoint=True)
    rs = np.random.RandomState(2)
    T, S, R = 23, 5, 9
    snode, amp, wave = rs.randint(0, s.N, S), rs.uniform(0.5, 1.5, S), rs.standard_normal((T, S))
    snode[1] = snode[0]                                   # two sources on one node
    snode[2] = int(np.flatnonzero(flags)[0])              # one on a wall
    rnode = rs.randint(0, s.N, R)
    rnode[1] = rnode[0]                                   # two receivers on one node
    rnode[2] = snode[0]
    grad = torch.tensor(rs.standard_normal((T, R)), device="cuda", dtype=s.cdtype)
    eps0 = torch.tensor(1 + rs.uniform(size=s.N), device="cuda", dtype=s.cdtype)

    def gradients(S2, R2):
        pad = rs.randint(0, s.N, max(S2 - S, 0)), rs.randint(0, s.N, max(R2 - R, 0))
        prob = AdjointProblem(s, T, np.r_[snode, pad[0]], np.c_[wave, np.zeros((T, S2 - S))], np.r_[rnode, pad[1]], ckpt_every=4)
        eps = eps0.clone().requires_grad_(True)
        a = torch.tensor(np.r_[amp, np.zeros(S2 - S)], device="cuda", dtype=s.cdtype).requires_grad_(True)
        tr = MaxwellFn.apply(eps, a, prob)
        tr.backward(torch.cat([grad, torch.zeros((T, R2 - R), device="cuda", dtype=s.cdtype)], 1))
        return tr[:, :R].detach(), eps.grad, a.grad[:S]

    few = gradients(S, R)
    assert all(float(g.abs().max()) > 0 for g in few)
    for S2, R2 in ((16, 64), (17, R), (S, 65), (17, 65), (40, 300)):
        for a, b in zip(gradients(S2, R2), few):
            assert torch.equal(a, b), (S2, R2)
