"""The permittivity of a differentiable run is one value per node: anything else is
refused before a kernel reads it (a column used to be refused by the copy to the
host, and its gradient could not have been returned)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import AdjointProblem, MaxwellFn, Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


@pytest.mark.parametrize("shape", [lambda n: (n, 1), lambda n: (1, n), lambda n: (n + 1,), lambda n: (2 * n,), lambda n: (n // 2,),
                                   lambda n: ()])
def test_other_shapes_are_refused(shape):
    xyz, flags, h = nodes.jittered_grid((16, 14), seed=3)
    s = Solver(2, xyz, flags, h, 12, 2, 2, 1e-4 / (configs.SC * h), (0.0,) * 2, (1.0,) * 2, precision="f32", adjoint=True)
    prob = AdjointProblem(s, 4, np.array([40]), np.ones((4, 1)), np.array([41, 42]))
    amp = torch.ones(1, device="cuda")
    good = torch.full((s.N,), 1.5, device="cuda", requires_grad=True)
    MaxwellFn.apply(good, amp, prob).sum().backward()
    assert good.grad.shape == good.shape
    with pytest.raises(ValueError):
        MaxwellFn.apply(torch.full(shape(s.N), 1.5, device="cuda", requires_grad=True), amp, prob)
