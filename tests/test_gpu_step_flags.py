"""Runs in whole steps that may be in flight together share no flags: what one run
leaves in the plan's memory or the workspace, the next does not touch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2508_18205_amd import Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402


@pytest.mark.parametrize("shape", [(16, 16), (16, 17), (200, 200)])
def test_runs_have_flags_of_their_own(shape):
    xyz, flags, h = nodes.jittered_grid(shape, seed=3)
    s = Solver(2, xyz, flags, h, 25, 2, 2, 1e-4 / (configs.SC * h), (0.0,) * 2, (1.0,) * 2, precision="f32")
    s.set_variant(block=256, xcd=1, lds=1)
    rs = np.random.RandomState(1)
    st = s.state(rs.standard_normal(s.N), rs.standard_normal((s.N, 2)))

    def memory():
        return torch.cat([s.arena[:s.arena.numel() // 8 * 8], s.ws[:1 << 20]]).view(torch.int64)

    # three tags (run, step) that no two runs have in common, one for each of the tiles
    was, touched = memory(), []
    for T in (3, 4, 3):
        s.run(st, T)
        now = memory()
        touched.append(was != now)
        was = now
    tiles = -(-s.N // 256)
    assert [int(t.sum()) for t in touched] == [tiles] * 3
    assert not bool((touched[0] & touched[1]).any() | (touched[1] & touched[2]).any() | (touched[0] & touched[2]).any())
