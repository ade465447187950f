"""Workloads that say what a user of the library waits for.

Every case is one pass of a program that keeps its plan (node set, weights on
the GPU) and its initial fields: a simulation from those fields, a gradient, a
hyperviscosity search, or a set-up of a new node set.  Sizes and method
parameters are those of this repository's workloads (51^2 cavities, the
40k-node dispersion study, 10^6-node pulses, 3D cubes, the K = 64 batch, the
250k-node inverse problem) and the range between them; node sets are jittered
grids, and the fields are smooth modes and pulses, as in those workloads.

``exact`` advances the same problem in 64 bits with its own stencils, weights
and steps.
"""
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2508_18205_amd import AdjointProblem, MaxwellFn, Solver, State

SC = 1.0 / (10.0 * math.sqrt(2.0))          # Courant number of every run of the method's paper
_DTYPE = {"f64": torch.float64, "f32": torch.float32}


def listed():
    return [
        # the paper-sized cavity: 2601 nodes, one period of its lowest mode; launches and latency are all there is
        dict(name="cavity_f64", kind="run", dim=2, sides="51x51", bc="PEC", pol="TM", n=12, m=2, alpha=2, chat=1e-3,
             precision="f64", weights="", T=1000, energy_every=100, rcv=0, src=0, tune=True),
        # the same cavity with E and H on two node sets
        dict(name="twoset_f64", kind="run", dim=2, sides="51x51", bc="PEC", pol="TM", n=12, m=2, alpha=2, chat=1e-3,
             precision="f64", weights="", T=400, energy_every=0, rcv=0, src=0, tune=True, twoset=True),
        # the dispersion study: periodic 200^2, wide stencils, E sampled on a line of 200 nodes
        dict(name="dispersion_f32", kind="run", dim=2, sides="200x200", bc="PERIODIC", pol="TM", n=60, m=2, alpha=2,
             chat=1.7e-5, precision="f32", weights="", T=300, energy_every=20, rcv=200, src=0, tune=True),
        # the headline pulse: 10^6 nodes, fourth-order curl, Delta^3 hyperviscosity
        dict(name="pulse_f32", kind="run", dim=2, sides="1000x1000", bc="PEC", pol="TM", n=25, m=4, alpha=3, chat=1e-4,
             precision="f32", weights="", T=20, energy_every=0, rcv=0, src=0, tune=True),
        # a ragged set in full precision, the other polarisation, the untuned default variant
        dict(name="te_f64", kind="run", dim=2, sides="613x401", bc="PEC", pol="TE", n=25, m=2, alpha=2, chat=1e-4,
             precision="f64", weights="", T=20, energy_every=10, rcv=0, src=0, tune=False),
        # the 3D cube at 10^6 nodes
        dict(name="cube_f32", kind="run", dim=3, sides="100x100x100", bc="PEC", pol="TM", n=35, m=2, alpha=2, chat=1e-3,
             precision="f32", weights="", T=10, energy_every=0, rcv=0, src=0, tune=True),
        # a small ragged 3D box in full precision with a source and receivers
        dict(name="box_f64", kind="run", dim=3, sides="31x23x19", bc="PEC", pol="TM", n=35, m=2, alpha=2, chat=1e-3,
             precision="f64", weights="", T=60, energy_every=0, rcv=8, src=1, tune=False),
        # 64 shots on one node set
        dict(name="batch64_f32", kind="batch", sides="500x500", n=25, m=2, alpha=2, chat=1e-4, K=64, T=10),
        # hyperviscosity search at the size of the dispersion study
        dict(name="hv_scan_f32", kind="scan", sides="200x200", n=25, m=2, alpha=2, K=16, T=400, energy_every=20, rounds=1),
        # gradient of 16 receiver traces with respect to the permittivity: forward and backward
        dict(name="gradient_f32", kind="adjoint", sides="500x500", n=25, m=2, alpha=2, chat=1e-4, precision="f32", T=100,
             rcv=16),
        # a new node set: reorder, stencils, local systems, packing, then two steps on it
        dict(name="setup2d_f32", kind="setup", dim=2, sides="400x400", n=25, m=4, alpha=3, chat=1e-4, precision="f32", T=2),
        dict(name="setup3d_f64", kind="setup", dim=3, sides="45x45x45", n=35, m=2, alpha=2, chat=1e-3, precision="f64", T=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(("run2d", "run2d", "run2d", "run3d", "twoset", "batch", "scan", "adjoint", "setup"))
    prec = rng.choice(("f32", "f32", "f64"))
    n, m, alpha = rng.choice(((12, 2, 2), (13, 2, 2), (20, 2, 2), (25, 2, 2), (30, 2, 2), (31, 4, 2), (25, 4, 3), (60, 2, 2)))
    if kind == "run2d":
        a = _log_int(rng, 40, 900)
        b = max(24, int(a * rng.uniform(0.5, 1.1)))
        bc = rng.choice(("PEC", "PEC", "PERIODIC"))
        pol = rng.choice(("TM", "TM", "TE"))
        w22 = prec == "f32" and rng.random() < 0.3
        probes = pol == "TM" and rng.random() < 0.6
        return dict(kind="run", dim=2, sides=f"{a}x{b}", bc=bc, pol=pol, n=n, m=m, alpha=alpha,
                    chat=rng.choice((1e-4, 1e-3)), precision=prec, weights="w22" if w22 else "",
                    T=max(11, min(301, int(6e6 / (a * b)))), energy_every=rng.choice((0, 10, 25)),
                    rcv=_log_int(rng, 1, 200) if probes else 0, src=rng.choice((0, 1, 3)) if probes else 0,
                    tune=rng.random() < 0.6)
    if kind == "twoset":
        a = _log_int(rng, 30, 500)
        return dict(kind="run", dim=2, sides=f"{a}x{a}", bc="PEC", pol="TM", n=rng.choice((12, 25)), m=2, alpha=2,
                    chat=1e-3, precision=prec, weights="", T=max(10, min(200, int(3e6 / (a * a)))),
                    energy_every=rng.choice((0, 10)), rcv=0, src=0, tune=rng.random() < 0.6, twoset=True)
    if kind == "run3d":
        a = _log_int(rng, 12, 90)
        b, c = (max(10, int(a * rng.uniform(0.6, 1.1))) for _ in range(2))
        probes = rng.random() < 0.5
        return dict(kind="run", dim=3, sides=f"{a}x{b}x{c}", bc=rng.choice(("PEC", "PEC", "PERIODIC")), pol="TM", n=35, m=2,
                    alpha=2, chat=1e-3, precision=prec, weights="", T=max(8, min(100, int(2e6 / (a * b * c)))),
                    energy_every=rng.choice((0, 5)), rcv=_log_int(rng, 1, 40) if probes else 0, src=int(probes),
                    tune=rng.random() < 0.6)
    if kind == "batch":
        a = _log_int(rng, 60, 480)
        return dict(kind="batch", sides=f"{a}x{max(50, int(a * rng.uniform(0.6, 1.0)))}", n=rng.choice((12, 25, 31)), m=2, alpha=2,
                    chat=1e-4, K=rng.choice((4, 8, 16, 32, 64)), T=rng.randint(6, 20))
    if kind == "scan":
        a = _log_int(rng, 60, 250)
        return dict(kind="scan", sides=f"{a}x{a - rng.randint(0, 9)}", n=rng.choice((12, 25)), m=2, alpha=2,
                    K=rng.choice((8, 16, 32, 64)), T=rng.randint(100, 300), energy_every=10, rounds=1)
    if kind == "adjoint":
        a = _log_int(rng, 60, 480)
        return dict(kind="adjoint", sides=f"{a}x{max(50, int(a * rng.uniform(0.6, 1.0)))}", n=rng.choice((12, 25)), m=2, alpha=2,
                    chat=1e-4, precision=prec, T=rng.randint(40, 120), rcv=_log_int(rng, 1, 64))
    if rng.random() < 0.5:
        a = _log_int(rng, 40, 400)
        return dict(kind="setup", dim=2, sides=f"{a}x{max(24, int(a * rng.uniform(0.6, 1.0)))}", n=n, m=m, alpha=alpha, chat=1e-4,
                    precision=prec, T=2)
    a = _log_int(rng, 11, 44)
    return dict(kind="setup", dim=3, sides=f"{a}x{max(10, a - rng.randint(0, 5))}x{max(10, a - rng.randint(0, 5))}", n=35, m=2,
                alpha=2, chat=1e-3, precision=prec, T=2)


# ---- problems: nodes, walls, parameters, initial fields ----------------------

def _grid(sides, lo, hi, periodic, rs):
    """Jittered grid (+-h/4 per axis; wall nodes stay on their wall): nodes [N, d] (x fastest), flags, h."""
    d = len(sides)
    idx = np.stack([g.transpose(tuple(reversed(range(d)))).reshape(-1)
                    for g in np.meshgrid(*[np.arange(s) for s in sides], indexing="ij")], axis=1)
    xyz = np.empty(idx.shape)
    flags = np.zeros(len(idx), np.uint8)
    for k in range(d):
        hk = (hi[k] - lo[k]) / (sides[k] if periodic else sides[k] - 1)
        x = lo[k] + hk * (idx[:, k] + rs.uniform(-0.25, 0.25, len(idx)))
        if periodic:
            x = lo[k] + np.mod(x - lo[k], hi[k] - lo[k])
            x[x >= hi[k]] = lo[k]
        else:
            a, b = idx[:, k] == 0, idx[:, k] == sides[k] - 1
            x[a], x[b] = lo[k], hi[k]
            flags |= (a * np.uint8(1 << (2 * k))) | (b * np.uint8(2 << (2 * k)))
        xyz[:, k] = x
        if k == 0:
            h = hk
    return xyz, flags, h


def _problem(case, seed):
    """Everything of a case that does not depend on the library."""
    rs = np.random.RandomState(seed % (1 << 32))
    sides = tuple(int(s) for s in case["sides"].split("x"))
    d = len(sides)
    periodic = case.get("bc") == "PERIODIC" or case["kind"] == "scan"
    step = 1.0 / (sides[0] if periodic else sides[0] - 1)
    lo, hi = (0.0,) * d, tuple(step * (s if periodic else s - 1) for s in sides)
    xyz, flags, h = _grid(sides, lo, hi, periodic, rs)
    N, alpha = len(xyz), case["alpha"]
    p = dict(dim=d, sides=sides, lo=lo, hi=hi, periodic=periodic, xyz=xyz, flags=flags, h=h, n=case["n"], m=case["m"],
             alpha=alpha, n_hv=2 * math.comb(2 * alpha + d, d) + 1, dt=SC * h, pol=case.get("pol", "TM"), N=N)
    p["hv_c"] = case.get("chat", 1e-4) / p["dt"]
    xh = xyz
    if case.get("twoset"):
        hsides = tuple(s - 1 for s in sides)
        iy, ix = np.meshgrid(np.arange(hsides[1]), np.arange(hsides[0]), indexing="ij")
        g = np.stack([ix.reshape(-1), iy.reshape(-1)], axis=1)
        xh = h * (g + 0.5 + rs.uniform(-0.25, 0.25, g.shape))
        p.update(xyz_h=xh, hsides=hsides)
    # a pulse around a drawn centre plus a smooth wave with drawn phases
    L = np.array(hi)
    c = L * rs.uniform(0.3, 0.7, d)
    width = max(4.0 * h, 0.06)

    def smooth(x, count):
        f = np.empty((len(x), count))
        for j in range(count):
            ph = rs.uniform(0, 2 * math.pi, d)
            f[:, j] = 0.3 * np.prod(np.cos(2 * math.pi * x / L + ph), axis=1)
        return f

    fe = 3 if d == 3 else (2 if p["pol"] == "TE" else 1)
    fh = 3 if d == 3 else (1 if p["pol"] == "TE" else 2)
    E0 = smooth(xyz, fe) + np.exp(-((xyz - c) ** 2).sum(1) / width ** 2)[:, None]
    E0 *= _keep(p, fe)
    p.update(fe=fe, fh=fh, E0=E0, H0=smooth(xh, fh))
    if case["kind"] == "scan":
        p["E0"] = p["E0"] + 1e-3 * rs.standard_normal(p["E0"].shape)
    if case["kind"] == "batch":
        p["centres"] = L * rs.uniform(0.2, 0.8, (case["K"], d))
        p["width"] = max(4.0 * h, 20.0 / 500)
    T = case["T"]
    if case.get("src") or case["kind"] == "adjoint":
        S = case.get("src") or 1
        inner = np.flatnonzero(flags == 0)
        t = (np.arange(T) + 0.5) * p["dt"]
        tau = max(T * p["dt"] / 8, 4 * p["dt"])
        p["src"] = (rs.choice(inner, S, replace=False), rs.uniform(0.5, 1.5, S),
                    np.stack([np.exp(-((t - (2 + s) * tau) / tau) ** 2) for s in range(S)], axis=1))
    if case.get("rcv"):
        if periodic and d == 2 and case["rcv"] <= sides[0]:
            p["rcv"] = (sides[1] // 2) * sides[0] + np.arange(case["rcv"])      # nodes along a line
        else:
            p["rcv"] = rs.choice(N, case["rcv"], replace=False)
    if case["kind"] == "adjoint":
        # receivers sit around the source, where the traces are not zero within the run
        s = p["src"][0][0]
        order = np.argsort(((xyz - xyz[s]) ** 2).sum(1), kind="stable")
        p["rcv"] = rs.choice(order[1:1 + 8 * case["rcv"]], case["rcv"], replace=False)
        p["eps"] = 1.0 + 0.5 * np.prod(np.cos(3 * math.pi * xyz / L + rs.uniform(0, 2 * math.pi, d)), axis=1) ** 2
        p["data"] = 0.1 * rs.standard_normal((T, case["rcv"]))
    return p


def _keep(p, fe):
    """[N, fe] factors of the conducting walls (0 = a component tangential to a wall)."""
    k = np.ones((p["N"], fe))
    if p["periodic"]:
        return k
    f = p["flags"]
    if fe == 1:
        k[f != 0] = 0
    else:
        for axis in range(p["dim"]):
            for comp in range(fe):
                if comp != axis:
                    k[(f & (3 << (2 * axis))) != 0, comp] = 0
    return k


def _solver(p, precision, **kw):
    if "xyz_h" in p:
        kw.update(mode="STAG2", xyz_h=p["xyz_h"], h_h=p["h"])
    return Solver(p["dim"], p["xyz"], p["flags"], p["h"], p["n"], p["m"], p["alpha"], p["hv_c"], p["lo"], p["hi"],
                  n_hv=p["n_hv"], bc="PERIODIC" if p["periodic"] else "PEC", pol=p["pol"], precision=precision, **kw)


# ---- the passes ------------------------------------------------------------------

def prepare(case, seed):
    p = _problem(case, seed)
    kind = case["kind"]
    g = dict(case=case, p=p)
    if kind == "setup":
        return g
    if kind == "run":
        s = _solver(p, case["precision"], weights=case["weights"] or None)
        st = s.state(p["E0"], p["H0"])
        if case["tune"]:
            s.autotune(st, reps=10)
        st = s.state(p["E0"], p["H0"])
        g.update(s=s, st=st, E0=st.E.clone(), H0=st.H.clone())
    elif kind == "batch":
        s = _solver(p, "f32", K=case["K"])
        x = torch.tensor(p["xyz"], device="cuda")
        c = torch.tensor(p["centres"], device="cuda")
        r2 = ((x[:, None, :] - c[None]) ** 2).sum(2)
        E = s.permute(torch.exp(-r2 / p["width"] ** 2).float().reshape(p["N"], 1, case["K"]).contiguous())
        H = torch.zeros((p["N"], 2, case["K"]), dtype=torch.float32, device="cuda")
        g.update(s=s, st=State([E, torch.zeros_like(E)], [H, torch.zeros_like(H)]), E0=E.clone(), H0=H.clone())
    elif kind == "scan":
        s = _solver(p, "f32", K=case["K"])
        E = torch.zeros((p["N"], 1, case["K"]), dtype=torch.float32, device="cuda")
        H = torch.zeros((p["N"], 2, case["K"]), dtype=torch.float32, device="cuda")
        g.update(s=s, st=State([E, torch.zeros_like(E)], [H, torch.zeros_like(H)]))
    elif kind == "adjoint":
        s = _solver(p, case["precision"], adjoint=True)
        dt = _DTYPE[case["precision"]]
        g.update(s=s, prob=AdjointProblem(s, case["T"], p["src"][0], p["src"][2], p["rcv"]),
                 eps=torch.tensor(p["eps"], dtype=dt, device="cuda"), amp=torch.tensor(p["src"][1], dtype=dt, device="cuda"),
                 data=torch.tensor(p["data"], dtype=dt, device="cuda"))
    return g


def _fields(s, st, twoset=False):
    """The current E and H in the caller's node order, on the GPU."""
    return {"E": s.permute(st.E, 0, False), "H": s.permute(st.H, 1 if twoset else 0, False)}


def run(g):
    case, p, kind = g["case"], g["p"], g["case"]["kind"]
    if kind == "run":
        s, st = g["s"], g["st"]
        st.E.copy_(g["E0"])
        st.H.copy_(g["H0"])
        r = s.run(st, case["T"], energy_every=case["energy_every"], src=p.get("src"), rcv=p.get("rcv"), use_graph=True)
        out = _fields(s, st, "xyz_h" in p)
        out.update({k: r[k] for k in ("energy", "traces") if k in r})
        return out
    if kind == "batch":
        s, st = g["s"], g["st"]
        st.E.copy_(g["E0"])
        st.H.copy_(g["H0"])
        s.step(st, case["T"])
        return _fields(s, st)
    if kind == "scan":
        lo, hi = _bracket(p)
        r = g["s"].hv_scan(g["st"], p["E0"], p["H0"], lo, hi, case["rounds"], case["T"], case["energy_every"], _BAND)
        return {k: r[k] for k in ("c", "ok", "umin", "umax")}
    if kind == "adjoint":
        eps, amp = g["eps"].clone().requires_grad_(True), g["amp"].clone().requires_grad_(True)
        tr = MaxwellFn.apply(eps, amp, g["prob"])
        (0.5 * ((tr - g["data"]) ** 2).sum()).backward()
        return {"traces": tr.detach(), "grad_eps": eps.grad, "grad_amp": amp.grad}
    s = _solver(p, case["precision"])
    st = s.state(p["E0"], p["H0"])
    s.step(st, case["T"])
    return _fields(s, st)


_BAND = (0.9, 1.02)


def _bracket(p):
    return 1e-6 / p["dt"], 1e-3 / p["dt"]


def work(case):
    """Bytes and operations of one pass, each weight, index, field read or written once per half step."""
    sides = [int(s) for s in case["sides"].split("x")]
    d, N = len(sides), math.prod(sides)
    n, nh = case["n"], 2 * math.comb(2 * case["alpha"] + d, d) + 1
    K, T = case.get("K", 1), case["T"]
    sw = 8 if case.get("precision") == "f64" else (3 if case.get("weights") == "w22" else 4)
    sf = 8 if case.get("precision") == "f64" else 4
    F = 3 if d == 2 else 6
    pairs = (n - 1) * (4 if d == 2 else 12) + (nh - 1) * F                 # products of one step, one field
    step = N * (2 * ((d * (n - 1) + nh - 1) * sw + 2 * (nh - 1)) + 3 * F * sf * K)   # 2-byte positions
    steps = T
    if case["kind"] == "scan":
        steps = T * case["rounds"]
    if case["kind"] == "adjoint":
        steps = 3 * T                                                       # forward, recomputation, reverse
    w = {"bytes": float(step * steps), "flops": float(2 * pairs * N * K * steps)}
    if case["kind"] == "setup":
        solve = sum((a + math.comb(b + d, d)) ** 3 * 2 / 3 for a, b in ((n, case["m"]), (nh, 2 * case["alpha"])))
        w["flops"] += N * solve
        w["bytes"] += float(N * ((d * n + nh) * (8 + sw) + 6 * nh))
    return w


# ---- the same problems in 64 bits -----------------------------------------------

def _nearest(p, centres, sides, src, k, centre_grid):
    """[C, k] nearest nodes of the jittered grid ``src`` (nodes of grid ``sides``) to the centres, whose own grid cells
    are ``centre_grid`` [C, d] in units of that grid, nearest first."""
    d = len(sides)
    full = (k / (math.pi if d == 2 else 4.1888)) ** (1.0 / d)
    reach = int(math.ceil(full + 1.0)) if p["periodic"] else int(math.ceil(2 * full + 1.0))   # a corner sees a quarter (an eighth)
    reach = min(reach, max(sides))
    off = np.stack(np.meshgrid(*[np.arange(-reach, reach + 1)] * d, indexing="ij"), -1).reshape(-1, d)
    off = off[(off ** 2).sum(1) <= (reach + 0.5) ** 2 * (1 if p["periodic"] else d)]
    mul = np.cumprod([1] + list(sides[:-1]))
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    tsrc, toff = torch.tensor(src, device=dev), torch.tensor(off, device=dev)
    S, M = torch.tensor(sides, device=dev), torch.tensor(mul, device=dev)
    P = torch.tensor([h - l for l, h in zip(p["lo"], p["hi"])], device=dev)
    out = np.empty((len(centres), k), np.int64)
    rows = max(1, int(3e7 / len(off)))
    for b in range(0, len(centres), rows):
        g = torch.tensor(centre_grid[b:b + rows], device=dev)[:, None, :] + toff[None]
        bad = torch.zeros(g.shape[:2], dtype=torch.bool, device=dev)
        if p["periodic"]:
            g = torch.remainder(g, S)
        else:
            bad = ((g < 0) | (g >= S)).any(2)
            g = torch.minimum(g.clamp(min=0), S - 1)
        ids = (g * M).sum(2)
        dx = tsrc[ids] - torch.tensor(centres[b:b + rows], device=dev)[:, None, :]
        if p["periodic"]:
            dx = dx - P * torch.round(dx / P)
        d2 = (dx * dx).sum(2)
        d2[bad] = math.inf
        near = d2.topk(k, dim=1, largest=False, sorted=True).indices
        out[b:b + rows] = ids.gather(1, near).cpu().numpy()
    return out


def _exponents(d, m):
    if d == 2:
        return [(g - b, b) for g in range(m + 1) for b in range(g + 1)]
    return [(a, b, g - a - b) for g in range(m + 1) for a in range(g + 1) for b in range(g - a + 1)]


def _weights(p, centres, src, idx, phs, m, alpha):
    """Weights at every centre: the d first derivatives (alpha = 0) or Delta^alpha, [C, ops, k]."""
    d = p["dim"]
    exps = _exponents(d, m)
    P = np.array([h - l for l, h in zip(p["lo"], p["hi"])])
    C, k = idx.shape
    ops = 1 if alpha else d
    W = np.empty((C, ops, k))
    lap = 1.0
    for j in range(alpha):
        lap *= (phs - 2 * j) * (phs - 2 * j + d - 2)
    rhs_p = np.zeros((len(exps), ops))
    for q, e in enumerate(exps):
        if alpha:
            if sum(e) == 2 * alpha and not any(x % 2 for x in e):
                rhs_p[q, 0] = math.factorial(alpha) / math.prod(math.factorial(x // 2) for x in e) * math.prod(
                    math.factorial(x) for x in e)
        elif sum(e) == 1:
            rhs_p[q, e.index(1)] = 1.0

    def rows(b):
        ix = idx[b:b + 256]
        x = src[ix] - centres[b:b + 256, None, :]
        if p["periodic"]:
            x = x - P * np.round(x / P)
        s = np.sqrt((x * x).sum(2)).max(1)
        x = x / s[:, None, None]
        R = k + len(exps)
        A = np.zeros((len(ix), R, R))
        r2 = sum((x[:, :, None, a] - x[:, None, :, a]) ** 2 for a in range(d))
        A[:, :k, :k] = np.sqrt(r2) * r2 ** (phs // 2)
        mono = np.stack([math.prod([x[..., a] ** e[a] for a in range(d)]) for e in exps], 2)
        A[:, :k, k:] = mono
        A[:, k:, :k] = mono.transpose(0, 2, 1)
        r = np.sqrt((x * x).sum(2))
        B = np.empty((len(ix), R, ops))
        B[:, k:] = rhs_p
        if alpha:
            B[:, :k, 0] = lap * r ** (phs - 2 * alpha)
        else:
            B[:, :k] = -phs * r[..., None] ** (phs - 2) * x
        w = np.linalg.solve(A, B)[:, :k]
        W[b:b + 256] = w.transpose(0, 2, 1) / (s ** (2 * alpha if alpha else 1))[:, None, None]

    with ThreadPoolExecutor(8) as ex:
        list(ex.map(rows, range(0, C, 256)))
    return W


class _Exact:
    """Stencils, weights and the leapfrog in 64 bits."""

    def __init__(self, p):
        self.p = p
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        d, sides = p["dim"], p["sides"]
        cell = np.stack([np.arange(p["N"]) // m % s for m, s in zip(np.cumprod([1] + list(sides[:-1])), sides)], 1)
        ch = 2 * p["alpha"] + 1
        if "xyz_h" in p:
            hs = p["hsides"]
            cell_h = np.stack([np.arange(len(p["xyz_h"])) // m % s for m, s in zip((1, hs[0]), hs)], 1)
            e, h = (p["xyz"], sides, cell), (p["xyz_h"], hs, cell_h)
            self.op_h, self.op_e = self._op(h, e, ch), self._op(e, h, ch)
        else:
            e = (p["xyz"], sides, cell)
            self.op_h = self.op_e = self._op(e, e, ch)
        self.a = p["dt"]
        self.gamma0 = (-1.0) ** (p["alpha"] - 1) * p["h"] ** (2 * p["alpha"])
        self.keep = torch.tensor(_keep(p, p["fe"]), device=self.dev)

    def _op(self, centre, other, phs_hv):
        """Curl weights on the other set's nodes, hyperviscosity weights on the own ones."""
        p = self.p
        t = lambda v: torch.tensor(v, device=self.dev)  # noqa: E731
        ic = _nearest(p, centre[0], other[1], other[0], p["n"], centre[2])
        ih = _nearest(p, centre[0], centre[1], centre[0], p["n_hv"], centre[2])
        wc = _weights(p, centre[0], other[0], ic, 3, p["m"], 0)
        wh = _weights(p, centre[0], centre[0], ih, phs_hv, 2 * p["alpha"], p["alpha"])
        return t(ic), t(wc), t(ih), t(wh[:, 0])

    @staticmethod
    def apply(w, idx, f):
        """sum_s w_s f_s for f [N] or [N, K]."""
        return (w * f[idx]).sum(1) if f.dim() == 1 else torch.stack([(w * c[idx]).sum(1) for c in f.unbind(1)], 1)

    def curl(self, op, f, sign):
        """The scheme's curl of the other field's components (list) in each polarisation; sign: of the vector form."""
        dd = [lambda v, k=k: self.apply(op[1][:, k], op[0], v) for k in range(self.p["dim"])]
        if self.p["dim"] == 3:
            return [dd[1](f[2]) - dd[2](f[1]), dd[2](f[0]) - dd[0](f[2]), dd[0](f[1]) - dd[1](f[0])]
        if len(f) == 1:
            return [dd[1](f[0]), -dd[0](f[0])]
        return [dd[0](f[1]) - dd[1](f[0])]

    def step(self, E, H, kappa, gamma, add=None):
        """One leapfrog step; E and H are lists of components."""
        hv = lambda op, f: self.apply(op[3], op[2], f)  # noqa: E731
        Hn = [h - self.a * (c - gamma * hv(self.op_h, h)) for h, c in zip(H, self.curl(self.op_h, E, 1))]
        En = [e + kappa * (c + gamma * hv(self.op_e, e)) for e, c in zip(E, self.curl(self.op_e, Hn, 1))]
        if add is not None:
            En[-1] = En[-1].index_add(0, add[0], add[1])
        En = [e * (self.keep[:, j] if e.dim() == 1 else self.keep[:, j, None]) for j, e in enumerate(En)]
        return En, Hn

    def energy(self, E, H, Hn):
        v = self.p["h"] ** self.p["dim"]
        return v * (sum((e * e).sum(0) for e in E) + sum((0.25 * (a + b) ** 2).sum(0) for a, b in zip(H, Hn)))


def exact(case, seed):
    sides = [int(s) for s in case["sides"].split("x")]
    d, N, kind = len(sides), math.prod(sides), case["kind"]
    R = 2 * math.comb(2 * case["alpha"] + d, d) + 1 + math.comb(2 * case["alpha"] + d, d)
    if N * R ** 3 > 1.6e11 or (kind == "adjoint" and N * case["T"] > 2.6e7):
        return None                                  # the local systems (the stored steps) alone take too long
    p = _problem(case, seed)
    x = _Exact(p)
    t = lambda v: torch.tensor(v, dtype=torch.float64, device=x.dev)  # noqa: E731
    E, H = list(t(p["E0"]).unbind(1)), list(t(p["H0"]).unbind(1))
    gamma = p["hv_c"] * x.gamma0

    def outputs(E, H):
        pad = lambda f: torch.stack(f + [torch.zeros_like(f[0])] * (d == 3), 1)  # noqa: E731
        return {"E": pad(E), "H": pad(H)}

    if kind == "batch":
        r2 = ((t(p["xyz"])[:, None, :] - t(p["centres"])[None]) ** 2).sum(2)
        E = [torch.exp(-r2 / p["width"] ** 2).float().double()]
        H = [torch.zeros_like(E[0]), torch.zeros_like(E[0])]
        for _ in range(case["T"]):
            E, H = x.step(E, H, x.a, gamma)
        return outputs(E, H)
    if kind == "scan":
        lo, hi = _bracket(p)
        K, res = case["K"], {"c": [], "ok": [], "umin": [], "umax": []}
        for _ in range(case["rounds"]):
            c = lo * (hi / lo) ** (np.arange(K) / (K - 1))
            g = t(c) * x.gamma0
            Ek = [f.float().double()[:, None].expand(-1, K) for f in E]
            Hk = [f.float().double()[:, None].expand(-1, K) for f in H]
            u = []
            for n in range(case["T"]):
                En, Hn = x.step(Ek, Hk, x.a, g)
                if n % case["energy_every"] == 0:
                    u.append(x.energy(Ek, Hk, Hn))
                Ek, Hk = En, Hn
            u = (torch.stack(u) / u[0]).cpu().numpy()
            bad = ~np.isfinite(u).all(0)
            umin, umax = u.min(0), np.where(bad, np.inf, u.max(0))
            ok = ~bad & (umin >= _BAND[0]) & (umax <= _BAND[1])
            for k, v in (("c", c), ("umin", umin), ("umax", umax)):
                res[k].append(v)
            if not ok.any() or ok[0]:
                break
            k = int(np.argmax(ok))
            lo, hi = c[k - 1], c[k]
        return {"c": np.array(res["c"]), "ok": None, "umin": np.array(res["umin"]), "umax": np.array(res["umax"])}
    if kind == "adjoint":
        f = _DTYPE[case["precision"]]
        eps = t(p["eps"]).to(f).double().requires_grad_(True)
        amp = t(p["src"][1]).to(f).double().requires_grad_(True)
        node, wave = torch.tensor(p["src"][0], device=x.dev), t(p["src"][2])
        rcv = torch.tensor(p["rcv"], device=x.dev)
        E, H, tr = [0 * eps], [torch.zeros_like(eps.detach())] * 2, []

        def one(E, Hx, Hy, eps, amp, w):
            En, Hn = x.step([E], [Hx, Hy], x.a / eps, gamma, (node, amp * w))
            return En[0], Hn[0], Hn[1]

        e, hx, hy = E[0], H[0], H[1]
        for n in range(case["T"]):
            e, hx, hy = torch.utils.checkpoint.checkpoint(one, e, hx, hy, eps, amp, wave[n], use_reentrant=False)
            tr.append(e[rcv])
        tr = torch.stack(tr)
        (0.5 * ((tr - t(p["data"]).to(f).double()) ** 2).sum()).backward()
        return {"traces": tr.detach(), "grad_eps": eps.grad, "grad_amp": amp.grad}
    energy, traces = [], []
    src = p.get("src") if kind == "run" else None
    every = case.get("energy_every", 0)
    for n in range(case["T"]):
        add = None
        if src is not None:
            add = (torch.tensor(src[0], device=x.dev), t(src[1] * src[2][n]))
        En, Hn = x.step(E, H, x.a, gamma, add)
        if every and n % every == 0:
            energy.append(x.energy(E, H, Hn))
        E, H = En, Hn
        if kind == "run" and "rcv" in p:
            traces.append(E[-1][torch.tensor(p["rcv"], device=x.dev)])
    out = outputs(E, H)
    if energy:
        out["energy"] = torch.stack(energy)
    if traces:
        out["traces"] = torch.stack(traces)
    return out
