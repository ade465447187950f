"""The register-resident local solver at the sizes where its register block
changes (32, 48, 64, 80, 96, 112 rows; 20, 36, 48, 64, 72, 88, 112 columns) and
just past it, on walled and periodic sets: weights against the oracle's LAPACK
solves, within its tests' bound for well-conditioned systems scaled by the
condition number; runs of graph-replayed steps against launched ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import knn, weights as ow  # noqa: E402
from paper_2508_18205_amd import Solver, _abi  # noqa: E402
from synth import nodes  # noqa: E402

EPS = np.finfo(float).eps


def _check(s, xyz, n, m, alpha, n_hv, period):
    p = s.perm
    idx = knn.knn(xyz, max(n, n_hv), period=period)
    for op, k, deg, phs, ref in (
            (_abi.OP_CURL_H, n, m, 3, lambda i: ow.curl_weights(xyz, xyz, i, m, period=period)),
            (_abi.OP_HV_H, n_hv, 2 * alpha, 2 * alpha + 1, lambda i: ow.hv_weights(xyz, xyz, i, alpha, period=period))):
        i = idx[:, :k]
        want = ref(i)[p].reshape(s.N, -1)
        got = s.weights(op).reshape(s.N, -1)
        cond = ow.system_condition(xyz, xyz, i, deg, phs, period)[p]
        err = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
        # two backward-stable eliminations of R unknowns: each within ~R eps cond, the pivot growth of random systems aside
        R = k + ow.n_monomials(xyz.shape[1], deg)
        assert np.all(err <= 4 * R * EPS * cond + 1e-14)


@pytest.mark.parametrize("n,m,alpha,n_hv", [
    (12, 2, 2, 31), (14, 2, 1, 17), (26, 2, 2, 33), (28, 2, 2, 34), (31, 4, 2, 46), (34, 3, 2, 49), (40, 4, 2, 50),
    (56, 2, 2, 57), (59, 3, 3, 60), (65, 4, 3, 67), (80, 5, 3, 69), (88, 2, 3, 83), (95, 2, 3, 84)])
@pytest.mark.parametrize("periodic", [False, True])
def test_solver_blocks_2d(n, m, alpha, n_hv, periodic):
    xyz, flags, h = nodes.jittered_grid((19, 17), seed=n, periodic=periodic)
    s = Solver(2, xyz, flags, h, n, m, alpha, 1.0, (0.0, 0.0), (1.0, 1.0), n_hv=n_hv, bc="PERIODIC" if periodic else "PEC")
    _check(s, xyz, n, m, alpha, n_hv, (1.0, 1.0) if periodic else None)


@pytest.mark.parametrize("n,m,alpha,n_hv", [(22, 2, 1, 25), (35, 2, 2, 71), (45, 3, 2, 76), (67, 3, 2, 77), (90, 2, 1, 99)])
def test_solver_blocks_3d(n, m, alpha, n_hv):
    xyz, flags, h = nodes.jittered_grid((8, 7, 9), seed=n)
    s = Solver(3, xyz, flags, h, n, m, alpha, 1.0, (0.0,) * 3, (1.0,) * 3, n_hv=n_hv)
    _check(s, xyz, n, m, alpha, n_hv, None)


@pytest.mark.parametrize("T", [191, 192, 193, 259])
def test_graph_stretches(T):
    """Runs on both sides of the length from which graphs replay the steps, with and without samples, eager steps between."""
    rs = np.random.RandomState(T)
    xyz, flags, h = nodes.jittered_grid((21, 19), seed=3, periodic=True)
    s = Solver(2, xyz, flags, h, 12, 2, 2, 1e-3, (0.0, 0.0), (1.0, 1.0), bc="PERIODIC")
    E0, H0 = rs.standard_normal((s.N, 1)), rs.standard_normal((s.N, 2))
    res = []
    for graph in (False, True):
        st = s.state(E0, H0)
        s.run(st, T, use_graph=graph)
        s.step(st, 3)
        en = s.run(st, T + 200, energy_every=T + 5, use_graph=graph)["energy"]
        res.append((st.E.clone(), st.H.clone(), en))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1]) and np.array_equal(res[0][2], res[1][2])
