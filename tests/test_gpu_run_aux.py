"""What rbffd_run does beside the bare steps -- sources and receivers folded
into the half-step kernels, samples and checkpoints launched where they are
due -- at the counts where a branch changes: 16 sources are the most the E
update looks through per node, several sources share a node, receivers
outnumber a small grid's threads and repeat, N is odd (checkpoint parts that
are multiples of 4 or 8 bytes only), T ends on and beside a sample."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import setup as osetup, step as ostep  # noqa: E402
from paper_2508_18205_amd import Solver  # noqa: E402
from synth import configs, nodes  # noqa: E402

# FP64 runs of a few steps differ from the oracle's only by summation order on weights that agree to ~1e-12
# (the GPU's own set-up); FP32 ones by at most the bar every FP32 test of this library uses
TOL = {"f64": 1e-10, "f32": 1e-5}


def _workload(dim, T, S, R, seed=3):
    rs = np.random.RandomState(seed)
    if dim == 2:
        xyz, flags, h = nodes.jittered_grid((23, 17), seed=seed)                  # N = 391
        w = configs.Workload("aux", 2, xyz, flags, h, 12, 2, 2, 31, 1e-3, T)
        w.E0, w.H0 = rs.standard_normal((w.N, 1)), rs.standard_normal((w.N, 2))
    else:
        xyz, flags, h = nodes.jittered_grid((7, 9, 11), seed=seed)                # N = 693
        w = configs.Workload("aux", 3, xyz, flags, h, 35, 2, 2, 71, 1e-3, T, lo=(0.0,) * 3, hi=(1.0,) * 3)
        w.E0, w.H0 = rs.standard_normal((w.N, 3)), rs.standard_normal((w.N, 3))
    w.E0[flags != 0] = 0.0
    w.src_node = rs.randint(0, w.N, S)
    w.src_node[-1] = w.src_node[0]                        # two sources on one node
    w.src_node[S // 2] = int(np.flatnonzero(flags)[0])    # one on a wall
    w.src_amp = rs.uniform(0.5, 1.5, S)
    w.src_wave = rs.standard_normal((T, S))
    w.rcv_node = rs.randint(0, w.N, R)
    w.rcv_node[:S] = w.src_node[:R]
    return w


@pytest.mark.parametrize("dim,precision,T,S,R,lds", [
    (2, "f64", 7, 1, 1, 1), (2, "f64", 6, 16, 700, 3), (2, "f64", 7, 17, 5, 0), (2, "f32", 7, 16, 65, 1),
    (2, "f64", 1, 3, 64, 1), (3, "f64", 7, 16, 33, 1), (3, "f64", 6, 17, 1500, 0), (3, "f32", 5, 3, 17, 1)])
def test_run_auxiliaries(dim, precision, T, S, R, lds):
    w = _workload(dim, T, S, R)
    oh, oe = osetup.operators(w)
    Eo, Ho, eno, tro = osetup.run_workload(w, oh, oe, energy_every=3)
    s = Solver.from_workload(w, precision=precision)
    s.set_variant(block=256, xcd=1, lds=lds)
    st = s.state(w.E0, w.H0)
    out = s.run(st, T, energy_every=3, src=(w.src_node, w.src_amp, w.src_wave), rcv=w.rcv_node, ckpt_every=2)
    tol = TOL[precision]
    scale = np.abs(tro).max()
    assert np.abs(out["traces"].cpu().numpy() - tro).max() <= tol * scale
    assert ostep.rel_l2(s.E_original(st), Eo) <= tol and ostep.rel_l2(s.H_original(st), Ho) <= tol
    assert np.abs(out["energy"] - eno).max() <= tol * np.abs(eno).max()
    # checkpoint k holds the state after 2 k steps, bit for bit
    ck, slot = out["ckpt"], s.sizes.e_bytes + s.sizes.h_bytes
    for k in range((T + 1) // 2):
        a = s.state(w.E0, w.H0)
        if k:
            s.run(a, 2 * k, src=(w.src_node, w.src_amp, w.src_wave))
        got = ck[k * slot:(k + 1) * slot]
        assert torch.equal(got[:s.sizes.e_bytes], a.E.contiguous().view(-1).view(torch.uint8))
        assert torch.equal(got[s.sizes.e_bytes:], a.H.contiguous().view(-1).view(torch.uint8))


@pytest.mark.parametrize("dim,precision,lds", [(2, "f32", 0), (2, "f32", 1), (2, "f32", 3), (2, "bf16", 1), (2, "f64", 3),
                                               (3, "f32", 0), (3, "f32", 1), (3, "f32", 3), (3, "f64", 2)])
def test_folded_sources_equal_separate(dim, precision, lds):
    # silent sources on far nodes make them 17: the same terms, added by a kernel of their own
    w = _workload(dim, 9, 5, 1)
    s = Solver.from_workload(w, precision=precision)
    s.set_variant(block=256, xcd=1, lds=lds)
    out = []
    for pad in (0, 12):
        st = s.state(w.E0, w.H0)
        s.run(st, 9, src=(np.r_[w.src_node, np.zeros(pad, int)], np.r_[w.src_amp, np.zeros(pad)],
                          np.c_[w.src_wave, np.zeros((9, pad))]))
        out.append((st.E.clone(), st.H.clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("K", [4, 24, 64, 80])
def test_batch_energy_samples(K):
    """Per-field energies of a batch at odd widths against the sum of eq. 20 over the stored fields."""
    rs = np.random.RandomState(K)
    xyz, flags, h = nodes.jittered_grid((31, 27), seed=4)
    s = Solver(2, xyz, flags, h, 12, 2, 2, 1e-3 / (configs.SC * h), (0.0, 0.0), (1.0, 1.0), n_hv=31, precision="f32", K=K)
    E0, H0 = rs.standard_normal((K, s.N, 1)), rs.standard_normal((K, s.N, 2))
    st = s.state_batched(E0, H0)
    en = s.run(st, 5, energy_every=2)["energy"]
    ref = []
    st = s.state_batched(E0, H0)
    for n in range(5):
        E, H = st.E.double(), st.H.double()
        s.step(st, 1)
        if n % 2 == 0:
            Hb = 0.5 * (H + st.H.double())
            ref.append(h * h * ((E * E).sum((0, 1)) + (Hb * Hb).sum((0, 1))))
    ref = torch.stack(ref).cpu().numpy()
    assert en.shape == ref.shape and np.abs(en / ref - 1).max() <= 1e-12     # FP64 sums of ~2500 terms
