"""A run in whole steps recorded into the caller's own HIP graph: every replay, with
eager runs of the same plan and synchronisations between, gives the eager result."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


@pytest.mark.parametrize("T", [1, 2, 5])
@pytest.mark.parametrize("patience", [5000, 0])
def test_replays_equal_eager(T, patience):
    xyz, flags, h = nodes.jittered_grid((120, 110), seed=3)
    s = Solver(2, xyz, flags, h, 25, 2, 2, 1e-4 / (configs.SC * h), (0.0,) * 2, (1.0,) * 2, precision="f32")
    s.set_variant(block=256, xcd=1, lds=1)
    s.set_patience(patience)
    assert s.whole_steps()["whole"]
    rs = np.random.RandomState(T)
    st = s.state(rs.standard_normal(s.N), rs.standard_normal((s.N, 2)))
    other = s.state(rs.standard_normal(s.N), rs.standard_normal((s.N, 2)))
    start, cur = (st.E.clone(), st.H.clone()), st.cur

    def passes(advance):                                  # each goes on from the fields of the one before
        E, H = start
        out = []
        for _ in range(4):
            st.cur = cur
            st.E.copy_(E), st.H.copy_(H)
            advance()
            torch.cuda.synchronize()
            st.cur = cur ^ (T & 1)
            E, H = st.E.clone(), st.H.clone()
            out.append((E, H))
            s.run(other, 3)
            torch.cuda.synchronize()
        return out

    eager = passes(lambda: s.run(st, T))
    st.cur = cur
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.run(st, T)
    for (E, H), (Ee, He) in zip(passes(g.replay), eager):
        assert torch.equal(E, Ee) and torch.equal(H, He)
