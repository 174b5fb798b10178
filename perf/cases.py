"""Performance cases of lesjet: the calls its users make, with inputs, work and 64-bit results.

A case names a mesh, a model and a call:

  mesh      "jet"       cylindrical jet mesh (30 D long, 20 D wide, lip-line clustering; no
                        node on the axis), entrance, exit, cross-axis, far field
            "jet_node"  the same with mesh nodes on the axis (centerline condition)
            "box"       periodic Cartesian box, 2 pi wide
            "wavy"      periodic non-orthogonal mesh (every metric term varies in 3-D)
  sgs       0 none, 1 Smagorinsky, 2 Vreman, 3 dynamic Smagorinsky
  precision "fp64" or "fp32" (FP32 storage of stage states and metrics)
  schedule  0 everything per RK stage, 1 viscosities and boundary values once per step
  call      "residual", "step" (`steps` RK5 steps under the CFL condition), "vjp" (residual
            VJP), "step_vjp" (VJP of one RK5 step of fixed dt), "diagnostics" (totals and
            azimuthal statistics)

`exact` is a plain torch statement of the same method in 64 bits (the VJPs by torch autograd).
"""
import math

import numpy as np
import torch

from paper_2301_00817_amd.solver import Solver

GAMMA = 1.4
ALPHA = (1.0 / 4.0, 1.0 / 6.0, 3.0 / 8.0, 1.0 / 2.0, 1.0)
DEV = "cuda" if torch.cuda.is_available() else "cpu"
UJ, UCO, THETA = 1.4, 0.05, 0.05      # jet and coflow Mach numbers, momentum thickness / D


def _case(name, call, mesh, nx, nr, nth, sgs=1, precision="fp64", schedule=0, steps=1):
    c = dict(call=call, mesh=mesh, nx=nx, nr=nr, nth=nth, sgs=sgs, precision=precision,
             schedule=schedule, steps=steps)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # smallest calls: one residual and one step of the 32^3 vortex box, where launches and
        # latency are what a user waits for (parity runs, restarts, coupling loops)
        _case("residual_box32", "residual", "box", 32, 32, 32),
        _case("step_box32", "step", "box", 32, 32, 32),
        # time marching of the 5.9 M-point jet, the ordinary production mesh, in both forms
        _case("step_jet6M", "step", "jet", 288, 160, 128, steps=2),
        _case("step_jet6M_fp32", "step", "jet", 288, 160, 128, precision="fp32", steps=2),
        # the paper's mesh C as the paper ran it (no subgrid model), FP32 storage
        _case("step_meshC_fp32", "step", "jet", 256, 256, 360, sgs=0, precision="fp32"),
        # the largest: one step of the 102 M-point jet
        _case("step_jet102M", "step", "jet", 800, 400, 320),
        # a general curvilinear mesh of odd size: residual of an implicit or verification driver
        _case("residual_wavy95", "residual", "wavy", 95, 95, 95),
        # axis-node centerline, Vreman, the paper's update order, ragged sizes
        _case("step_node_vreman", "step", "jet_node", 173, 67, 90, sgs=2, schedule=1, steps=2),
        # dynamic model, coefficients from every stage state
        _case("step_dynamic", "step", "jet", 160, 100, 128, sgs=3),
        # reverse mode on the 2 M-point jet: residual VJP and RK5-step VJP (gradient rollouts)
        _case("vjp_jet2M", "vjp", "jet", 160, 100, 128),
        _case("step_vjp_jet2M", "step_vjp", "jet", 160, 100, 128),
        # totals and azimuthal statistics between steps
        _case("diagnostics_jet6M", "diagnostics", "jet", 288, 160, 128),
    ]


def draw(rng):
    call = rng.choice(["residual", "step", "step", "vjp", "step_vjp", "diagnostics"])
    adjoint = call in ("vjp", "step_vjp")
    mesh = rng.choice(["jet", "jet", "jet", "jet_node", "box", "wavy"])
    sgs = rng.choice([0, 1, 1, 2] if adjoint or mesh == "jet_node" else [0, 1, 1, 2, 3])
    precision = "fp64" if adjoint else rng.choice(["fp64", "fp32"])
    points = math.exp(rng.uniform(math.log(2e4), math.log(3e6 if adjoint or sgs == 3 else 8e6)))
    # three lengths around the cube root, odd ones included; the jets need an even azimuth
    a, b = rng.uniform(0.6, 1.7), rng.uniform(0.6, 1.4)
    s = points ** (1.0 / 3.0)
    nx, nr = max(9, round(s * a)), max(9, round(s * b))
    nth = max(10, round(points / (nx * nr)))
    if mesh in ("jet", "jet_node"):
        nth += nth % 2
    if mesh == "wavy":
        nx = nr = nth = max(13, round(s))
    return _case(None, call, mesh, nx, nr, nth, sgs=sgs, precision=precision,
                 schedule=rng.choice([0, 0, 1]) if call == "step" else 0,
                 steps=rng.choice([1, 2]) if call == "step" else 1)


# ---- inputs ---------------------------------------------------------------------------------
def _params(case):
    jet = case["mesh"].startswith("jet")
    L = 2.0 * math.pi
    bc = ("periodic",) * 6
    if jet:
        bc = ("inflow", "outflow", "axis_node" if case["mesh"] == "jet_node" else "axis",
              "farfield", "periodic", "periodic")
    visc = UJ / 1.5e6 if jet else (1e-3 if case["sgs"] == 3 else 0.5 / 1.0e4)
    return dict(gamma=GAMMA, Pr=0.72, Pr_sgs=0.9, visc_coef=visc, suth_S=110.4 / 288.15,
                Cs=0.148, k2=0.25, k4=0.016, cfl=0.5, rk_alpha=ALPHA,
                ref_prim=(1.0, UCO if jet else 0.0, 0.0, 0.0, 1.0 / GAMMA), p_exit=1.0 / GAMMA,
                sgs_model=case["sgs"], schedule=case["schedule"], bc=bc,
                period=((0.0,) * 3,) * 3 if jet else ((L, 0, 0), (0, L, 0), (0, 0, L)))


def _maps(case):
    """Axial, radial and azimuthal node positions of a jet mesh: spacing growing by 1.005 along
    x, point density 1 + 50 sech^2((r - 0.5)/0.2) along r."""
    nx, nr, nth = case["nx"], case["nr"], case["nth"]
    x = 1.005 ** np.arange(nx) - 1.0
    X = 30.0 * x / x[-1]
    r0 = 0.0 if case["mesh"] == "jet_node" else 0.005
    fine = np.linspace(r0, 20.0, 200001)
    arc = fine + 50.0 * 0.2 * np.tanh((fine - 0.5) / 0.2)
    R = np.interp(np.linspace(arc[0], arc[-1], nr), arc, fine)
    R[0], R[-1] = r0, 20.0
    TH = 2.0 * math.pi * np.arange(nth) / nth
    return X, R, TH


def _coords(case, device):
    nx, nr, nth = case["nx"], case["nr"], case["nth"]
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=device)  # noqa: E731
    if case["mesh"].startswith("jet"):
        X, R, TH = _maps(case)
        X, R = t(X).view(1, 1, nx), t(R).view(1, nr, 1)
        ct = t([math.cos(a) for a in TH]).view(nth, 1, 1)
        st = t([math.sin(a) for a in TH]).view(nth, 1, 1)
        return torch.stack([v.expand(nth, nr, nx) for v in (X, R * ct, R * st)])
    L = 2.0 * math.pi
    x = (t(np.arange(nx)) * (L / nx)).view(1, 1, nx)
    y = (t(np.arange(nr)) * (L / nr)).view(1, nr, 1)
    z = (t(np.arange(nth)) * (L / nth)).view(nth, 1, 1)
    a = 0.1 if case["mesh"] == "wavy" else 0.0
    parts = (x + a * torch.sin(y), y + a * torch.sin(z), z + a * torch.sin(x)) if a else (x, y, z)
    return torch.stack([v.expand(nth, nr, nx) for v in parts])


def _conserved(rho, u, v, w, p):
    return torch.stack([rho, rho * u, rho * v, rho * w,
                        p / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v + w * w)])


def _profile(case, device):
    """Jet velocity u(r), (nr,)."""
    r = torch.as_tensor(_maps(case)[1], dtype=torch.float64, device=device)
    return UCO + 0.5 * (UJ - UCO) * (1.0 + torch.tanh((0.5 - r) / (2.0 * THETA)))


def _inputs(case, seed, device=DEV):
    """Interior state (5, nth, nr, nx), entrance target (5, nth, nr) or None, cotangent."""
    nx, nr, nth = case["nx"], case["nr"], case["nth"]
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed))
    noise = lambda *s: 2.0 * torch.rand(s, dtype=torch.float64, device=device, generator=gen) - 1.0  # noqa: E731
    one = torch.ones((nth, nr, nx), dtype=torch.float64, device=device)
    shape, inflow = (nth, nr, nx), None
    if case["mesh"].startswith("jet"):
        u2 = _profile(case, device).view(1, nr, 1)
        Q = _conserved(one * (1 + 1e-3 * noise(*shape)), u2 + 1e-3 * UJ * noise(*shape),
                       1e-3 * UJ * noise(*shape), 1e-3 * UJ * noise(*shape),
                       (one + 1e-3 * noise(*shape)) / GAMMA)
        uin = _profile(case, device).view(1, nr).expand(nth, nr)
        sp = (nth, nr)
        inflow = torch.stack([1 + 1e-3 * noise(*sp), uin + 1e-3 * UJ * noise(*sp),
                              1e-3 * UJ * noise(*sp), 1e-3 * UJ * noise(*sp),
                              (1 + 1e-3 * noise(*sp)) / GAMMA])
    else:
        x, y, z = _coords(case, device)
        if case["sgs"] == 3:       # a field with a decaying spectrum, on which the dynamic
            f = [0.0] * 4          # model's averages are well away from zero
            ph = torch.rand((4, 6), dtype=torch.float64, device=device, generator=gen) * 2 * math.pi
            for n, (a, b, c) in enumerate(((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (0, 2, 1), (2, 1, 1))):
                for m in range(4):
                    f[m] = f[m] + torch.cos(a * x + b * y + c * z + ph[m, n]) / (a * a + b * b + c * c)
            Q = _conserved(one, 0.1 * f[0], 0.1 * f[1], 0.1 * f[2], (1 + 0.05 * f[3]) / GAMMA)
        else:                      # isentropic Mach-0.5 vortex plus noise
            dx, dy = x - math.pi, y - math.pi
            c = 5.0 / (2.0 * math.pi * math.sqrt(GAMMA))
            e = torch.exp(0.5 * (1.0 - dx * dx - dy * dy))
            T = 1.0 - (GAMMA - 1.0) * 25.0 / (8.0 * GAMMA * math.pi ** 2) * e * e
            rho = T ** (1.0 / (GAMMA - 1.0))
            Q = _conserved(rho + 1e-4 * noise(*shape), 0.5 - c * dy * e + 1e-4 * noise(*shape),
                           c * dx * e + 1e-4 * noise(*shape), 1e-4 * noise(*shape),
                           rho * T / GAMMA + 1e-4 * noise(*shape))
    bar = noise(5, *shape) if case["call"] in ("vjp", "step_vjp") else None
    return Q, inflow, bar


def _dt(case):
    """Fixed time step of a step VJP: a fraction of the smallest cell's acoustic time."""
    if case["mesh"].startswith("jet"):
        X, R, TH = _maps(case)
        r = R[1] if case["mesh"] == "jet_node" else R[0]
        return 0.2 * min(r * (TH[1] - TH[0]), float(np.min(np.diff(R))), X[1]) / (UJ + 1.0)
    return 0.1 * 2.0 * math.pi / max(case["nx"], case["nr"], case["nth"])


def prepare(case, seed):
    Q, inflow, bar = _inputs(case, seed)
    if case["mesh"].startswith("jet"):
        mesh = dict(grid=tuple(torch.as_tensor(a) for a in _maps(case)))
    else:
        mesh = dict(xyz=_coords(case, "cuda"))
    s = Solver(_params(case), inflow=inflow, precision=case["precision"], device="cuda", **mesh)
    call = case["call"]
    st = dict(call=call, s=s, steps=case["steps"])
    if call == "residual":
        st["Q"], st["R"] = s.pad(Q), s.field(5)
    elif call == "step":
        st["Q"] = s.pad(Q, dtype=torch.float64)
        st["dt"] = torch.zeros(case["steps"], dtype=torch.float64, device="cuda")
    elif call in ("vjp", "step_vjp"):
        st["Q"], st["bar"] = s.pad(Q), s.pad(bar, fill=0.0)
        st["out"], st["h"] = s.field(5), _dt(case)
        st["inflow"] = inflow is not None
    else:
        st["Q"] = s.pad(Q, dtype=torch.float64)
    return st


def run(st):
    s, call = st["s"], st["call"]
    if call == "residual":
        return s.interior(s.residual(st["Q"], st["R"]))
    if call == "step":
        dt = s.rk5_step(st["Q"], st["steps"], 0.0, st["dt"])
        return {"Q": s.interior(st["Q"]), "dt": dt}
    if call == "diagnostics":
        s1, s2 = s.new_stats()
        return {"totals": s.diagnostics(st["Q"], (s1, s2)), "sum1": s1, "sum2": s2}
    ib = s.new_inflow_bar() if st["inflow"] else None
    if call == "vjp":
        s.residual_vjp(st["Q"], st["bar"], st["out"], inflow_bar=ib)
    else:
        s.rk5_step_vjp(st["Q"], st["h"], st["bar"], st["out"], inflow_bar=ib)
    return {"Qbar": s.interior(st["out"]), "inflow_bar": ib}


def work(case):
    """Per point: a residual reads and writes five variables and does about 1,200 operations (its
    VJP 3,000, reading Q and the cotangent); a stage also reads Q^n.  The wavy mesh has ten metric
    terms per point to read; on the others they follow from the one-dimensional node positions.
    A step VJP runs four stages and five residual VJPs; the dynamic model's coefficients take a
    further read of the state and 1,500 operations per evaluation."""
    n = case["nx"] * case["nr"] * case["nth"]
    ws = 4 if case["precision"] == "fp32" else 8
    met = 10 * ws if case["mesh"] == "wavy" else 0
    dyn_b, dyn_f = (5 * ws + met, 1500) if case["sgs"] == 3 else (0, 0)
    call = case["call"]
    if call == "residual":
        b, f = 10 * ws + met + dyn_b, 1200 + dyn_f
    elif call == "step":       # FP32 storage: Q^n and the returned state stay in FP64
        evals = 1 if case["schedule"] else 5
        b = case["steps"] * (5 * (10 * ws + 40 + met) + evals * dyn_b)
        f = case["steps"] * (5 * 1250 + evals * dyn_f)
    elif call == "vjp":
        b, f = 120 + met, 3000
    elif call == "step_vjp":
        b, f = 4 * (120 + met) + 5 * (120 + met), 4 * 1250 + 5 * 3000
    else:
        b, f = 40 + (8 if case["mesh"] == "wavy" else 0), 40
    return {"bytes": float(b * n), "flops": float(f * n)}


# ---- the same results in plain torch, 64 bits --------------------------------------------------
def exact(case, seed):
    n = case["nx"] * case["nr"] * case["nth"]
    call = case["call"]
    if n > 9e6:
        return None
    Q, inflow, bar = _inputs(case, seed)
    prm, geo = _params(case), _geometry(case)
    if call == "diagnostics":
        V = geo["V"][2:-2, 2:-2, 2:-2]
        rho, u, v, w, p = _prim(Q)
        f = torch.stack([rho, u, v, w, p])
        return {"totals": (V * Q).sum((1, 2, 3)), "sum1": f.sum(1), "sum2": (f * f).sum(1)}
    if call == "residual":
        if case["precision"] == "fp32":
            Q = Q.float().double()
        return _residual(Q, prm, geo, inflow)
    if call == "step":
        dts = []
        for _ in range(case["steps"]):
            Q, h = _step(Q, prm, geo, inflow)
            dts.append(h)
        if prm["bc"][2] == "axis_node":
            Q = _axis_mean(Q)
        return {"Q": Q, "dt": torch.stack(dts)}
    ib = torch.zeros_like(inflow) if inflow is not None else None

    def vjp(q, b):
        q = q.detach().requires_grad_(True)
        t = inflow.detach().requires_grad_(True) if inflow is not None else None
        g = torch.autograd.grad(_residual(q, prm, geo, t), (q, t) if t is not None else (q,), b,
                                allow_unused=True)
        return g[0], g[1] if t is not None else None

    if call == "vjp":
        qb, ib = vjp(Q, bar)
        return {"Qbar": qb, "inflow_bar": ib}
    h, X = _dt(case), [Q]
    for a in ALPHA[:4]:
        X.append(Q - a * h * _residual(X[-1], prm, geo, inflow))
    b = bar
    if prm["bc"][2] == "axis_node":
        q = torch.zeros_like(bar).requires_grad_(True)
        (b,) = torch.autograd.grad(_axis_mean(q), q, bar)
    out = b
    for a, q in zip(ALPHA[::-1], X[::-1]):
        b, g = vjp(q, -a * h * b)
        out = out + b
        ib = ib + g if ib is not None else None
    return {"Qbar": out, "inflow_bar": ib}


def _ext(A, lo, hi, dim):
    return torch.cat([lo, A, hi], dim)


def _geometry(case):
    """Area vectors S[d][m] and Jacobian V on the box padded by two points, from coordinates
    padded by three (wrapped, mirrored across the axis, or extrapolated) and central differences."""
    prm, P = _params(case), _coords(case, DEV)
    for d, dim in enumerate((3, 2, 1)):
        n = P.shape[dim]
        per = torch.tensor([float(v) for v in prm["period"][d]], dtype=torch.float64,
                           device=DEV).view(3, 1, 1, 1)
        at = lambda i: P.narrow(dim, i, 1)  # noqa: E731,B023
        kind = prm["bc"][2 * d]
        if kind == "periodic":
            lo = P.narrow(dim, n - 3, 3) - per
        elif kind in ("axis", "axis_node"):
            first = 0 if kind == "axis" else 1
            lo = torch.roll(P.narrow(2, first, 3).flip(2), case["nth"] // 2, 1)
        else:
            lo = torch.cat([at(0) + m * (at(0) - at(1)) for m in (3, 2, 1)], dim)
        if prm["bc"][2 * d + 1] == "periodic":
            hi = P.narrow(dim, 0, 3) + per
        else:
            hi = torch.cat([at(n - 1) + m * (at(n - 1) - at(n - 2)) for m in (1, 2, 3)], dim)
        P = _ext(P, lo, hi, dim)
    r = [_diff(P, d) for d in range(3)]                # r[d][c] = d x_c / d xi_d
    cross = lambda a, b: [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2],  # noqa: E731
                          a[0] * b[1] - a[1] * b[0]]
    S = [cross(r[1], r[2]), cross(r[2], r[0]), cross(r[0], r[1])]
    V = r[0][0] * S[0][0] + r[0][1] * S[0][1] + r[0][2] * S[0][2]
    return dict(S=S, V=V)


def _diff(A, d):
    """Central difference along direction d, one point shorter at every end."""
    n = [A.shape[-3] - 2, A.shape[-2] - 2, A.shape[-1] - 2]
    o = [[1, 1, 1], [1, 1, 1]]
    o[0][2 - d], o[1][2 - d] = 2, 0
    hi, lo = (A[..., a:a + n[0], b:b + n[1], e:e + n[2]] for a, b, e in o)
    return 0.5 * (hi - lo)


def _in(A, m=1):
    return A[..., m:-m, m:-m, m:-m]


def _prim(Q):
    rho = Q[0]
    u, v, w = Q[1] / rho, Q[2] / rho, Q[3] / rho
    return rho, u, v, w, (GAMMA - 1.0) * (Q[4] - 0.5 * rho * (u * u + v * v + w * w))


def _axis_mean(Q):
    m = Q[:, :, 1:2].mean(1, keepdim=True).expand(-1, Q.shape[1], -1, -1)
    return torch.cat([m, Q[:, :, 1:]], 2)


def _riemann(Q, out, n):
    """Boundary state from the Riemann invariants of the inside state Q and outside primitives."""
    e = _prim(Q)
    ae, ar = torch.sqrt(GAMMA * e[4] / e[0]), torch.sqrt(GAMMA * out[4] / out[0])
    qe = e[1] * n[0] + e[2] * n[1] + e[3] * n[2]
    qr = out[1] * n[0] + out[2] * n[1] + out[3] * n[2]
    rp, rm = qe + 2.0 * ae / (GAMMA - 1.0), qr - 2.0 * ar / (GAMMA - 1.0)
    qf, af = 0.5 * (rp + rm), 0.25 * (GAMMA - 1.0) * (rp - rm)
    leaving = qe >= 0
    s = [torch.where(leaving, a, b.expand_as(a)) for a, b in zip(e, out)]
    qs = torch.where(leaving, qe, qr)
    rho = (s[0] ** GAMMA * af * af / (GAMMA * s[4])) ** (1.0 / (GAMMA - 1.0))
    f = _conserved(rho, *(s[1 + m] + (qf - qs) * n[m] for m in range(3)), rho * af * af / GAMMA)
    o = _conserved(*(b.expand_as(qe) for b in out))
    M = qe / ae
    return torch.where(M >= 1.0, Q, torch.where(M <= -1.0, o, f))


def _unit(S, sl, sign):
    v = [a[sl] for a in S]
    return [sign * a / torch.sqrt(v[0] ** 2 + v[1] ** 2 + v[2] ** 2) for a in v]


def _fill(Q, prm, geo, inflow, held=None):
    """State with two ghost layers: xi, then eta, then zeta; held: a filled state whose physical
    faces and axis row are taken."""
    bc, nth = prm["bc"], Q.shape[1]
    node = bc[2] == "axis_node"
    if node:
        Q = torch.cat([held[:, 2:-2, 2:3, 2:-2], Q[:, :, 1:]], 2) if held is not None else _axis_mean(Q)
    two = lambda f, dim: torch.cat([f, f], dim)  # noqa: E731
    if bc[0] == "periodic":
        Q = _ext(Q, Q[..., -2:], Q[..., :2], 3)
    elif held is not None:
        Q = _ext(Q, held[:, 2:-2, 2:-2, :2], held[:, 2:-2, 2:-2, -2:], 3)
    else:
        def normal(i, sign):
            n = _unit(geo["S"][0], (slice(2, -2), slice(2, -2), i), sign)
            return [torch.cat([a[:, 1:2], a[:, 1:]], 1) for a in n] if node else n
        n = normal(2, -1.0)
        t = [inflow[c] for c in range(5)]
        sup = -(t[1] * n[0] + t[2] * n[1] + t[3] * n[2]) / torch.sqrt(GAMMA * t[4] / t[0]) >= 1.0
        lo = torch.where(sup, _conserved(*t), _riemann(Q[..., 0], t, n))[..., None]
        e, n = _prim(Q[..., -1]), normal(-3, 1.0)
        qn = e[1] * n[0] + e[2] * n[1] + e[3] * n[2]
        sub = _conserved(*e[:4], torch.full_like(e[4], prm["p_exit"]))
        hi = torch.where(qn / torch.sqrt(GAMMA * e[4] / e[0]) >= 1.0, Q[..., -1], sub)[..., None]
        Q = _ext(Q, two(lo, 3), two(hi, 3), 3)
    if bc[2] == "periodic":
        Q = _ext(Q, Q[:, :, -2:], Q[:, :, :2], 2)
    else:
        first = 1 if node else 0
        lo = torch.roll(Q[:, :, first:first + 2].flip(2), nth // 2, 1)
        if held is not None:
            hi = held[:, 2:-2, -2:]
        else:
            n = _unit(geo["S"][1], (slice(2, -2), -3), 1.0)
            ref = [torch.tensor(float(v), dtype=Q.dtype, device=Q.device) for v in prm["ref_prim"]]
            hi = two(_riemann(Q[:, :, -1], ref, n)[:, :, None], 2)
        Q = _ext(Q, lo, hi, 2)
    return _ext(Q, Q[:, -2:], Q[:, :2], 1)


def _filter(A):
    for dim in (-1, -2, -3):
        n = A.shape[dim] - 2
        A = 0.25 * A.narrow(dim, 0, n) + 0.5 * A.narrow(dim, 1, n) + 0.25 * A.narrow(dim, 2, n)
    return A


def _gradients(fields, S, V):
    """d phi / d x_m by the chain rule; S and V one point narrower than the fields."""
    out = []
    for phi in fields:
        dd = [_diff(phi, d) for d in range(3)]
        out.append([(S[0][m] * dd[0] + S[1][m] * dd[1] + S[2][m] * dd[2]) / V for m in range(3)])
    return out


def _strain(g):
    s = [[0.5 * (g[i][j] + g[j][i]) for j in range(3)] for i in range(3)]
    return s, 2.0 * sum(s[i][j] ** 2 for i in range(3) for j in range(3))


def _dynamic(Qp, prm, geo):
    """(C_I, C_ds, Pr_sgs) of the dynamic model: ratios of volume averages of test-filtered terms."""
    rho, u, v, w, p = _prim(Qp)
    T, vel = GAMMA * p / rho, (u, v, w)
    S1, V1 = [[_in(a) for a in r] for r in geo["S"]], _in(geo["V"])
    Si, Vi = [[_in(a) for a in r] for r in S1], _in(V1)
    g = _gradients((u, v, w, T), S1, V1)
    s, s2 = _strain(g)
    rS = _in(rho) * torch.sqrt(s2)
    D2 = Vi.abs() ** (2.0 / 3.0)
    fr, fru, frT = _filter(rho), [_filter(rho * a) for a in vel], _filter(rho * T)
    gh = _gradients([a / fr for a in fru] + [frT / fr], Si, Vi)
    sh, sh2 = _strain(gh)
    hr, hru, hrT, hS2 = _in(fr), [_in(a) for a in fru], _in(frT), _filter(_in(rho) * s2)
    s, gT = [[_in(a) for a in r] for r in s], [_in(a) for a in g[3]]
    trS, trSh = s[0][0] + s[1][1] + s[2][2], sh[0][0] + sh[1][1] + sh[2][2]
    hrSh = hr * torch.sqrt(sh2)
    Lll = LS = hSS = ShS = hSmm = 0.0
    for i in range(3):
        for j in range(3):
            Lij = _in(_filter(rho * vel[i] * vel[j])) - hru[i] * hru[j] / hr
            h = _filter(rS * 0.5 * (g[i][j] + g[j][i]))
            LS, hSS, ShS = LS + Lij * s[i][j], hSS + h * s[i][j], ShS + sh[i][j] * s[i][j]
            if i == j:
                Lll, hSmm = Lll + Lij, hSmm + h
    NP = sum(D2 * _filter(rS * g[3][j]) * gT[j] - 4.0 * D2 * hrSh * gh[3][j] * gT[j] for j in range(3))
    DP = sum((_in(_filter(rho * vel[j] * T)) - hru[j] * hrT / hr) * gT[j] for j in range(3))
    mean = lambda a: float((Vi * a).sum())  # noqa: E731
    DI = mean(8.0 * D2 * hr * sh2 - 2.0 * D2 * hS2)
    CI = max(mean(Lll) / DI, 0.0) if DI else 0.0
    Dd = mean(2.0 * D2 * (hSS - hSmm * trS / 3.0) - 8.0 * D2 * hrSh * (ShS - trSh * trS / 3.0))
    Cd = max((mean(LS - trS * Lll / 3.0) + CI * mean(2.0 * D2 * hS2 * trS / 3.0)) / Dd, 0.0) if Dd else 0.0
    dp = mean(DP)
    Pr = Cd * mean(NP) / dp if dp else math.nan
    return CI, Cd, Pr if math.isfinite(Pr) and Pr > 0.0 else prm["Pr_sgs"]


def _root(s2):
    """sqrt, with derivative 0 at 0 (the strain of the axis row)."""
    some = s2 > 0
    return torch.where(some, torch.sqrt(torch.where(some, s2, torch.ones_like(s2))), torch.zeros_like(s2))


def _points(Qp, prm, geo, held=None):
    """Point fluxes G[d], scaled spectral radii, sensors on [-1, n]^3 and the viscosities used."""
    S, V0 = [[_in(a) for a in r] for r in geo["S"]], _in(geo["V"])
    V = torch.where(V0 == 0.0, torch.ones_like(V0), V0)       # the axis row, whose values no face uses
    rho, u, v, w, p = _prim(Qp)
    T = GAMMA * p / rho
    q, pi = _in(Qp), _in(p)
    vel, Ti, ri = [_in(a) for a in (u, v, w)], _in(T), _in(rho)
    Uc = [S[d][0] * vel[0] + S[d][1] * vel[1] + S[d][2] * vel[2] for d in range(3)]
    Cv, sgs = prm["visc_coef"], prm["sgs_model"]
    g = _gradients((u, v, w, T), S, V)
    s, s2 = _strain(g)
    D2 = V.abs() ** (2.0 / 3.0)
    if held is None:
        mu = Ti ** 1.5 * (1.0 + prm["suth_S"]) / (Ti + prm["suth_S"])
        dyn, Prs = (0.0, 0.0, 0.0), prm["Pr_sgs"]
        mut = torch.zeros_like(mu)
        if sgs == 1:
            mut = ri * prm["Cs"] ** 2 * D2 * _root(s2) / Cv
        elif sgs == 2:
            b = [[g[i][0] * g[j][0] + g[i][1] * g[j][1] + g[i][2] * g[j][2] for j in range(3)] for i in range(3)]
            B = (b[0][0] * b[1][1] - b[0][1] ** 2 + b[0][0] * b[2][2] - b[0][2] ** 2
                 + b[1][1] * b[2][2] - b[1][2] ** 2)
            aa = b[0][0] + b[1][1] + b[2][2]
            ok = (aa > 0) & (B > 0)
            ratio = torch.sqrt(torch.where(ok, B, torch.ones_like(B)) / torch.where(ok, aa, torch.ones_like(B)))
            mut = torch.where(ok, ri * 2.5 * prm["Cs"] ** 2 * D2 * ratio / Cv, mut)
        elif sgs == 3:
            dyn = _dynamic(Qp, prm, geo)
            Prs = dyn[2]
            mut = ri * dyn[1] * D2 * torch.sqrt(s2) / Cv
        held = (mu + mut, (mu / prm["Pr"] + mut / Prs) / (GAMMA - 1.0), dyn)
    mt, kap, dyn = held
    pg = pi + (2.0 / 3.0) * dyn[0] * ri * D2 * s2 if sgs == 3 else pi
    div = g[0][0] + g[1][1] + g[2][2]
    tau = [[mt * (2.0 * s[i][j] - (2.0 / 3.0 * div if i == j else 0.0)) for j in range(3)] for i in range(3)]
    beta = [tau[0][j] * vel[0] + tau[1][j] * vel[1] + tau[2][j] * vel[2] + kap * g[3][j] for j in range(3)]
    G, nu = [], []
    for d in range(3):
        visc = [Cv * (S[d][0] * t[0] + S[d][1] * t[1] + S[d][2] * t[2]) for t in (*tau, beta)]
        G.append(torch.stack([ri * Uc[d]] + [q[1 + m] * Uc[d] + pg * S[d][m] - visc[m] for m in range(3)]
                             + [(q[4] + pg) * Uc[d] - visc[3]]))
        o = [slice(1, -1)] * 3
        hi, lo = list(o), list(o)
        hi[2 - d], lo[2 - d] = slice(2, None), slice(None, -2)
        pu, pl = p[tuple(hi)], p[tuple(lo)]
        nu.append((pu - 2.0 * pi + pl).abs() / (pu + 2.0 * pi + pl))
    if prm["bc"][2] == "axis_node":
        G[1] = torch.cat([G[1][:, :, :1], torch.zeros_like(G[1][:, :, :1]), G[1][:, :, 2:]], 2)
    a = torch.sqrt(Ti)
    norm = [torch.sqrt(r[0] ** 2 + r[1] ** 2 + r[2] ** 2) for r in S]
    # (the area of a face on the axis is zero: keep its root differentiable)
    norm = [torch.where(V0 == 0.0, torch.ones_like(m), m) for m in norm] if (V0 == 0.0).any() else norm
    lam = [(Uc[d].abs() + a * norm[d]) / V.abs() for d in range(3)]
    root = [torch.sqrt(m) for m in lam]
    return G, [m * (root[0] + root[1] + root[2]) for m in root], nu, held


def _residual(Q, prm, geo, inflow, held=None):
    Hp, visc = held if held is not None else (None, None)
    return _padded_residual(_fill(Q, prm, geo, inflow, Hp), prm, geo, visc)


def _padded_residual(Qp, prm, geo, visc):
    G, lb, nu, _ = _points(Qp, prm, geo, visc)
    W = torch.cat([Qp[:4], (Qp[4] + _prim(Qp)[4])[None]])
    V1, rhs = _in(geo["V"]), 0.0
    for d in range(3):
        dim = -1 - d

        def line(A, ng):
            for e in range(3):
                if e != d:
                    A = A.narrow(-1 - e, ng, A.shape[-1 - e] - 2 * ng)
            return A
        g, l, s, v, wl = line(G[d], 1), line(lb[d], 1), line(nu[d], 1), line(V1, 1), line(W, 2)
        nf = g.shape[dim] - 1
        cut = lambda A, o: A.narrow(dim, o, nf)  # noqa: E731,B023
        e2 = prm["k2"] * torch.maximum(cut(s, 0), cut(s, 1))
        e4 = torch.clamp(prm["k4"] - e2, min=0.0)
        lf, Vf = 0.5 * (cut(l, 0) + cut(l, 1)), 0.5 * (cut(v, 0) + cut(v, 1))
        Wm, WL, WR, Wp = (cut(wl, o) for o in range(4))
        d4 = Wp - 3.0 * WR + 3.0 * WL - Wm
        if d == 1 and prm["bc"][2] == "axis_node":      # face between the axis and row 1
            ax = torch.zeros(nf, dtype=torch.bool, device=Qp.device)
            ax[1] = True
            ax = ax.view(1, nf, 1)
            lf = torch.where(ax, cut(l, 1), lf)
            d4 = torch.where(ax, Wp - 4.0 * WR + 3.0 * WL, d4)
        keep = torch.ones(nf, dtype=torch.float64, device=Qp.device)
        for f, side in ((0, 0), (nf - 1, 1)):
            if prm["bc"][2 * d + side] in ("inflow", "outflow", "farfield"):
                keep[f] = 0.0
        keep = keep.view([nf if e == 2 - d else 1 for e in range(3)])
        F = 0.5 * (cut(g, 0) + cut(g, 1)) - keep * Vf * lf * (e2 * (WR - WL) - e4 * d4)
        rhs = rhs + F.narrow(dim, 1, nf - 1) - F.narrow(dim, 0, nf - 1)
    V = _in(V1)
    if prm["bc"][2] == "axis_node":
        r = rhs[:, :, 1:] / V[:, 1:]
        return torch.cat([torch.zeros_like(r[:, :, :1]), r], 2)
    return rhs / V


def _step(Q, prm, geo, inflow):
    rho, u, v, w, p = _prim(Q)
    a, tot = torch.sqrt(GAMMA * p / rho), 0.0
    first = 1 if prm["bc"][2] == "axis_node" else 0
    for d in range(3):
        S = [m[2:-2, 2:-2, 2:-2] for m in geo["S"][d]]
        tot = tot + (S[0] * u + S[1] * v + S[2] * w).abs() + a * torch.sqrt(S[0] ** 2 + S[1] ** 2 + S[2] ** 2)
    h = prm["cfl"] / (tot[:, first:] / geo["V"][2:-2, 2 + first:-2, 2:-2].abs()).max()
    held = None
    if prm["schedule"]:
        Hp = _fill(Q, prm, geo, inflow)
        held = (Hp, _points(Hp, prm, geo)[3])
    q = Q
    for al in ALPHA:
        q = Q - al * h * _residual(q, prm, geo, inflow, held)
    return q, h
