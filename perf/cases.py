"""The work that a user has this package do, as cases that can be timed and compared.

A case is one call (or one short sequence of calls) of the public entry points
of `paper_1607_06834_amd` on a seeded flow: one time step, a differentiated
trajectory, an adaptive integration, the operators f / J v / J^T w, a Krylov
basis, the stiffness estimate.  Flows, discretisations and Krylov dimensions
are those of the package's workloads (`rok_inputs.WORKLOADS`), of its adaptive
and eigenvalue runs on the cylinder grids, and ragged sizes between them.

`exact` is the same computation in plain torch, in double precision.
"""
import math

import torch

import rok_inputs as ri
from paper_1607_06834_amd import Rok
from paper_1607_06834_amd.autograd import rok_trajectory

GAMMA, PRANDTL = 1.4, 0.72
MACH_CYLINDER, MU_CYLINDER, SUTHERLAND = 0.3, 0.01, 0.4


def _case(call, flow, n, recon, jvp, M, **more):
    n = tuple(n) + (1,) * (3 - len(n))
    c = {"call": call, "flow": flow, "n0": n[0], "n1": n[1], "n2": n[2], "recon": recon, "flux": "rusanov",
         "jvp": jvp, "M": M, "precision": "fp64", "cfl": 2.0}
    c.update(more)
    return c


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)

    return [
        # the smallest workload: a 32^2 first-order vortex, 1024 cells, where launches and latency are all there is
        named("step_vortex32", "step", "vortex", (32, 32), "first", "fd", 8, cfl=5.0),
        # the cylinder runs: a viscous O-grid with thin wall cells, Roe's flux, Sutherland's law
        named("step_cylinder128x64", "step", "cylinder", (128, 64), "first", "fd", 8, flux="roe", h=2e-6),
        # an ordinary production grid whose sides are no multiples of anything
        named("step_vortex611x389", "step", "vortex", (611, 389), "muscl", "fd", 12),
        # the 1024^2 MUSCL vortex workload
        named("step_vortex1024", "step", "vortex", (1024, 1024), "muscl", "fd", 16, cfl=10.0),
        # the 2048^2 viscous Taylor-Green workload: f and J v in FP32, the Krylov part in FP64
        named("step_tgv2048_fp32", "step", "tgv", (2048, 2048), "muscl", "tangent", 20, precision="fp32", cfl=5.0),
        # a ragged 3-D grid in the precision form
        named("step_tgv90x75x61_fp32", "step", "tgv", (90, 75, 61), "muscl", "tangent", 16, precision="fp32", cfl=5.0),
        # the largest workload and the benchmark's: 256^3 viscous Taylor-Green, 84 M unknowns
        named("step_tgv256cubed", "step", "tgv", (256, 256, 256), "muscl", "fd", 16, cfl=10.0),
        # forward and backward: the gradient of the final kinetic energy through two 512^2 steps (the 50-step
        # workload repeats exactly this), every state a checkpoint
        named("gradient_vortex512", "gradient", "vortex", (512, 512), "first", "tangent", 16, steps=2),
        # adaptive integration with small bases, as in the work-precision runs
        named("adaptive_tgv512", "adaptive", "tgv", (512, 512), "muscl", "fd", 4, steps=3, tol=1e-5, cfl=4.0),
        # f, both products J v and J^T w on their own: what an outer solver of the user's own calls
        named("operators_tgv700x450", "operators", "tgv", (700, 450), "muscl", "both", 0),
        # a Krylov basis and its Hessenberg matrix with exact products, on a 3-D grid
        named("arnoldi_tgv64cubed", "arnoldi", "tgv", (64, 64, 64), "muscl", "tangent", 24),
        # the stiffness diagnostic on the cylinder grid
        named("eigs_cylinder128x64", "eigs", "cylinder", (128, 64), "first", "tangent", 40, flux="roe", k=6,
              restarts=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["step"] * 6 + ["gradient", "adaptive", "operators", "arnoldi", "eigs"])
    recon = rng.choice(["first", "muscl"])
    flux = rng.choice(["rusanov", "rusanov", "roe"])
    if call == "eigs":
        return _case("eigs", "cylinder", (_log_int(rng, 48, 160), _log_int(rng, 24, 80)), "first", "tangent",
                     rng.choice([24, 32, 40, 50]), flux=flux, k=rng.randint(2, 8), restarts=rng.randint(4, 10))
    if call == "gradient":
        return _case("gradient", "vortex", (_log_int(rng, 32, 512), _log_int(rng, 32, 512)), recon, "tangent",
                     rng.choice([4, 8, 12, 16]), steps=rng.randint(1, 2))
    if call == "adaptive":
        return _case("adaptive", rng.choice(["vortex", "tgv"]), (_log_int(rng, 32, 640), _log_int(rng, 32, 640)),
                     recon, "fd", rng.choice([0, 4, 8]), flux=flux, steps=rng.randint(1, 3),
                     tol=rng.choice([1e-4, 1e-5, 1e-6]), cfl=2.0)
    flow = rng.choice(["vortex", "tgv", "tgv3", "cylinder"] if call == "step" else ["vortex", "tgv", "tgv3"])
    if flow == "cylinder":
        return _case("step", "cylinder", (_log_int(rng, 48, 320), _log_int(rng, 24, 160)), recon, "fd",
                     rng.choice([4, 8, 12]), flux="roe", h=1e-6)
    if flow == "tgv3":
        flow, side = "tgv", _log_int(rng, 16, 160)
        n = [max(8, int(side * rng.uniform(0.7, 1.3))) for _ in range(3)]
        if rng.random() < 0.4:
            n = [16 * max(1, round(x / 16)) for x in n]
    else:
        side = _log_int(rng, 24, 1600)
        n = [max(8, int(side * rng.uniform(0.7, 1.3))) for _ in range(2)]
    if call == "operators":
        return _case("operators", flow, n, recon, "both", 0, flux=flux)
    if call == "arnoldi":
        return _case("arnoldi", flow, n, recon, "tangent", rng.randint(4, 24), flux=flux)
    jvp, precision = rng.choice([("fd", "fp64"), ("fd", "fp64"), ("tangent", "fp64"), ("tangent", "fp32")])
    return _case("step", flow, n, recon, jvp, rng.choice([0, 4, 8, 12, 16, 20]), flux=flux, precision=precision)


# ---------------------------------------------------------------------------
# Problems and seeded states, on the GPU
# ---------------------------------------------------------------------------

def _dims(case):
    return (case["n0"], case["n1"]) if case["n2"] == 1 else (case["n0"], case["n1"], case["n2"])


def _problem(case):
    """(problem, O-grid nodes or None)."""
    n = _dims(case)
    if case["flow"] == "cylinder":
        pb, nodes = ri.cylinder_ogrid(n[0], n[1], radius=0.5, far=20.0, recon=case["recon"], flux=case["flux"],
                                      cluster=10.0)
        return dict(pb, physics="ns", mu=MU_CYLINDER, sutherland=SUTHERLAND, t_ref=1.0), nodes
    if case["flow"] == "vortex":
        return ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", case["recon"], flux=case["flux"]), None
    L = 2.0 * math.pi
    return ri.problem(n, (0.0,) * len(n), (L,) * len(n), "ns", case["recon"], flux=case["flux"],
                      mu=1.0 / (100.0 if len(n) == 2 else 1600.0)), None


def _centres(pb, device):
    """Cell centres x, y(, z) as arrays indexed [z][y][x]."""
    cs = []
    for d, m in enumerate(pb["n"]):
        dx = (pb["hi"][d] - pb["lo"][d]) / m
        cs.append(pb["lo"][d] + (torch.arange(m, dtype=torch.float64, device=device) + 0.5) * dx)
    return torch.meshgrid(*reversed(cs), indexing="ij")[::-1]


def _state(case, pb, nodes, seed, device):
    """The flow with every primitive variable perturbed per cell by 0.1 % of its spread, as a flat conserved vector."""
    if case["flow"] == "cylinder":
        x, y = (torch.as_tensor(a, device=device) for a in nodes)
        c4 = lambda a: 0.25 * (a[:-1] + a[1:] + torch.roll(a, -1, 1)[:-1] + torch.roll(a, -1, 1)[1:])  # noqa: E731
        r = torch.sqrt(c4(x) ** 2 + c4(y) ** 2)
        u = MACH_CYLINDER * math.sqrt(GAMMA) * (1.0 - torch.exp(-(r - 0.5) / 0.1))   # a boundary layer at the wall
        q = [torch.ones_like(u), u, torch.zeros_like(u), torch.ones_like(u)]
    elif case["flow"] == "vortex":
        x, y = _centres(pb, device)
        uinf = 0.5 * math.sqrt(GAMMA) / math.sqrt(2.0)
        e = torch.exp(0.5 * (1.0 - (x * x + y * y)))
        b = 5.0 / (2.0 * math.pi)
        T = 1.0 - (GAMMA - 1.0) * b * b / (2.0 * GAMMA) * e * e
        rho = T ** (1.0 / (GAMMA - 1.0))
        q = [rho, uinf - b * y * e, uinf + b * x * e, rho * T]
    else:
        p0 = 1.0 / (GAMMA * 0.01)
        X = _centres(pb, device)
        if len(X) == 2:
            x, y = X
            q = [torch.ones_like(x), torch.sin(x) * torch.cos(y), -torch.cos(x) * torch.sin(y),
                 p0 + 0.25 * (torch.cos(2 * x) + torch.cos(2 * y))]
        else:
            x, y, z = X
            q = [torch.ones_like(x), torch.sin(x) * torch.cos(y) * torch.cos(z),
                 -torch.cos(x) * torch.sin(y) * torch.cos(z), torch.zeros_like(x),
                 p0 + (torch.cos(2 * x) + torch.cos(2 * y)) * (torch.cos(2 * z) + 2.0) / 16.0]
    gen = torch.Generator(device=device).manual_seed(seed)
    for m in range(len(q)):
        spread = float(q[m].max() - q[m].min())
        if spread < 1e-12:
            spread = max(1.0, float(q[m].abs().max())) * 0.1
        q[m] = q[m] + 1e-3 * spread * (2.0 * torch.rand(q[m].shape, generator=gen, dtype=torch.float64,
                                                        device=device) - 1.0)
    ke = sum(v * v for v in q[1:-1])
    return torch.stack([q[0]] + [q[0] * v for v in q[1:-1]] + [q[-1] / (GAMMA - 1.0) + 0.5 * q[0] * ke]).reshape(-1)


def _step_size(case, pb, y):
    """h = cfl / (max sum_d (|u_d| + c) / dx_d + max(nu) 4 sum_d dx_d^-2); the cylinder's is given."""
    if "h" in case:
        return case["h"]
    if case["flow"] == "cylinder":
        return 1e-6
    U = y.view((len(pb["n"]) + 2, -1))
    rho, vel = U[0], [m / U[0] for m in U[1:-1]]
    p = (GAMMA - 1.0) * (U[-1] - 0.5 * rho * sum(v * v for v in vel))
    c = torch.sqrt(GAMMA * p / rho)
    dx = [(pb["hi"][d] - pb["lo"][d]) / m for d, m in enumerate(pb["n"])]
    rate = float(sum((v.abs() + c) / dx[d] for d, v in enumerate(vel)).max())
    if pb["physics"] == "ns":
        rate += float((max(4.0 / 3.0, GAMMA / PRANDTL) * pb["mu"] / rho).max()) * 4.0 * sum(1.0 / a ** 2 for a in dx)
    return case["cfl"] / rate


def _freestream():
    return ri.freestream(mach=MACH_CYLINDER)


def _inputs(case, seed, device):
    pb, nodes = _problem(case)
    y = _state(case, pb, nodes, seed, device)
    gen = torch.Generator(device=device).manual_seed(seed + 1)
    v = w = None
    if case["call"] in ("operators", "eigs"):
        v, w = (torch.randn(y.numel(), generator=gen, dtype=torch.float64, device=device) for _ in range(2))
        v, w = v / v.norm(), w / w.norm()
    return pb, nodes, y, v, w, _step_size(case, pb, y)


def prepare(case, seed):
    pb, nodes, y, v, w, h = _inputs(case, seed, "cuda")
    rok = Rok(pb, case["precision"])
    if nodes is not None:
        rok.set_ogrid(*nodes, _freestream(), t_wall=1.0)
    tab = ri.rok4_tableau()
    if case["call"] == "step":
        rok.workspace(case["M"], tab["s"])   # a program that steps keeps one
    return {"case": case, "rok": rok, "y": y, "v": v, "w": w, "h": h, "tab": tab}


def run(state):
    c, rok, y, h, tab = (state[k] for k in ("case", "rok", "y", "h", "tab"))
    if c["call"] == "step":
        return rok.step(y, h, tab, c["M"], mode=c["jvp"])
    if c["call"] == "gradient":
        y0 = y.detach().requires_grad_(True)
        yk = rok_trajectory(rok, y0, h, tab, c["M"], c["steps"], checkpoint_every=1)
        (g,) = torch.autograd.grad(_kinetic_energy(yk), y0)
        return {"y": yk.detach(), "gradient": g}
    if c["call"] == "adaptive":
        yt, rec = rok.integrate_adaptive(y, c["steps"] * h, h, tab, c["M"], "fd", order=4, rtol=c["tol"],
                                         atol=c["tol"], max_steps=200)
        return {"y": yt, "accepted": rec["n_accepted"], "rejected": rec["n_rejected"]}
    if c["call"] == "operators":
        F = rok.residual(y)
        return {"f": F, "jv_fd": rok.jvp(y, state["v"], "fd", fy=F), "jv": rok.jvp(y, state["v"], "tangent"),
                "jtw": rok.vjp(y, state["w"])}
    if c["call"] == "arnoldi":
        V, H, m = rok.arnoldi(y, rok.residual(y), c["M"], "tangent")
        return {"V": V, "H": H, "m": m}
    values, _, restarts, converged = rok.eigs(y, state["v"], k=c["k"], m=c["M"], max_restarts=c["restarts"], tol=1e-8)
    return {"values": values, "restarts": restarts, "converged": converged}


def _kinetic_energy(y):
    """Sum over the cells of |m|^2 / (2 rho) of a 2-D state, over the number of cells."""
    U = y.view(4, -1)
    return (0.5 * (U[1] * U[1] + U[2] * U[2]) / U[0]).mean()


# ---------------------------------------------------------------------------
# The least work of a pass
# ---------------------------------------------------------------------------

def _f_flops(case):
    """Additions and multiplications of f per cell, divisions and roots counted as one each."""
    D = 2 if case["n2"] == 1 else 3
    nv = D + 2
    face = 2 * (4 * D + 8) + 6 * nv + (30 + 8 * nv if case["flux"] == "roe" else 0)
    if case["recon"] == "muscl":
        face += 2 * nv * 5 + 2 * (2 * D + 5)
    if case["flow"] != "vortex":
        face += 6 * D * D + 6 * D
    return D * (face + 2 * nv) + 3 * D + 6


def work(case):
    cells = case["n0"] * case["n1"] * case["n2"]
    N = (4 if case["n2"] == 1 else 5) * cells
    M, ff = case["M"], _f_flops(case) * cells
    s = 4
    product, dual = (4, 1) if case["jvp"] == "fd" else (3, 3)

    def basis(m):   # column j: the j + 1 basis vectors and w read, the next vector written; 4 flops per element and pass
        return sum(j + 3 for j in range(m)) + product * m, sum(4 * (j + 1) + 3 for j in range(m)) * N + dual * ff * m

    def step(m):    # f, the projection and the recovery of each stage, y in and y out
        b, f = basis(m)
        return b + s * (2 * m + 4) + 2, f + s * (ff + 6 * m * N)

    if case["call"] == "step":
        v, f = step(M)
    elif case["call"] == "gradient":   # the step and its recomputation, then its transpose, about twice the step
        v, f = step(M)
        v, f = 4 * case["steps"] * v, 4 * case["steps"] * f
    elif case["call"] == "adaptive":   # at least `steps` macro steps of three steps each would cover the interval
        v, f = step(M)
        v, f = 3 * case["steps"] * (v + 1), 3 * case["steps"] * f
    elif case["call"] == "operators":
        v, f = 2 + 4 + 3 + 3, (1 + 1 + 3 + 3) * ff
    elif case["call"] == "arnoldi":
        v, f = basis(M)
        v, f = v + 2, f + ff
    else:   # the first factorisation of m columns; restarts come on top
        v, f = basis(M)
    return {"bytes": 8.0 * N * v, "flops": float(f)}


# ---------------------------------------------------------------------------
# The same computations in plain torch, 64 bits
# ---------------------------------------------------------------------------

def _minmod(a, b):
    return torch.where(a * b <= 0, torch.zeros_like(a), torch.where(a.abs() <= b.abs(), a, b))


def _primitives(U):
    vel = U[1:-1] / U[0]
    return torch.cat([U[:1], vel, ((GAMMA - 1.0) * (U[-1] - 0.5 * U[0] * (vel * vel).sum(0)))[None]])


def _conserved(q):
    return torch.cat([q[:1], q[:1] * q[1:-1], (q[-1] / (GAMMA - 1.0) + 0.5 * q[0] * (q[1:-1] ** 2).sum(0))[None]])


def _euler(q, U, d):
    F = U * q[1 + d]
    return torch.stack([F[m] + q[-1] if m == 1 + d else (F[m] + q[-1] * q[1 + d] if m == len(q) - 1 else F[m])
                        for m in range(len(q))])


def _num_flux(flux, qL, qR, d):
    UL, UR = _conserved(qL), _conserved(qR)
    central = 0.5 * (_euler(qL, UL, d) + _euler(qR, UR, d))
    if flux == "rusanov":
        sL, sR = (q[1 + d].abs() + torch.sqrt(GAMMA * q[-1] / q[0]) for q in (qL, qR))
        return central - 0.5 * torch.maximum(sL, sR) * (UR - UL)
    # Roe's linearisation, Harten's fix of half-width c / 8 on the acoustic waves
    wl, wr = torch.sqrt(qL[0]), torch.sqrt(qR[0])
    u = (wl * qL[1:-1] + wr * qR[1:-1]) / (wl + wr)
    H = (wl * (UL[-1] + qL[-1]) / qL[0] + wr * (UR[-1] + qR[-1]) / qR[0]) / (wl + wr)
    rho, ke, dq = wl * wr, (u * u).sum(0), qR - qL
    c2 = (GAMMA - 1.0) * (H - 0.5 * ke)
    c, un, dun, dp = torch.sqrt(c2), u[d], dq[1 + d], dq[-1]
    fix = lambda lam: torch.where(lam.abs() < c / 8, (lam * lam + (c / 8) ** 2) / (c / 4), lam.abs())  # noqa: E731
    w1 = fix(un - c) * (dp - rho * c * dun) / (2 * c2)
    w2 = un.abs() * (dq[0] - dp / c2)
    w3 = fix(un + c) * (dp + rho * c * dun) / (2 * c2)
    rows = [w1 + w2 + w3]
    en = w1 * (H - un * c) + w2 * 0.5 * ke + w3 * (H + un * c)
    for e in range(u.shape[0]):
        shear = un.abs() * rho * dq[1 + e] if e != d else torch.zeros_like(un)
        rows.append((w1 + w2 + w3) * u[e] + (w3 - w1) * c * (1.0 if e == d else 0.0) + shear)
        if e != d:
            en = en + shear * u[e]
    return central - 0.5 * torch.stack(rows + [en])


def _f_box(case, pb):
    """y -> f(y) on the periodic box."""
    n, D = pb["n"], len(pb["n"])
    dx = [(pb["hi"][d] - pb["lo"][d]) / n[d] for d in range(D)]
    mu = pb["mu"]
    kappa = mu * GAMMA / ((GAMMA - 1.0) * PRANDTL)

    def f(y):
        q = _primitives(y.view((D + 2,) + tuple(reversed(n))))
        up = lambda a, d, k=1: torch.roll(a, -k, a.dim() - 1 - d)  # noqa: E731
        T = q[-1] / q[0]
        out = 0.0
        for d in range(D):
            if pb["recon"] == "muscl":
                s = _minmod(q - up(q, d, -1), up(q, d) - q)
                F = _num_flux(pb["flux"], q + 0.5 * s, up(q - 0.5 * s, d), d)
            else:
                F = _num_flux(pb["flux"], q, up(q, d), d)
            if pb["physics"] == "ns":
                v = q[1:-1]
                G = []   # G[b] = d(velocity)/dx_b at the face
                for b in range(D):
                    if b == d:
                        G.append((up(v, d) - v) / dx[d])
                    else:
                        g = (up(v, b) - up(v, b, -1)) * (0.5 / dx[b])
                        G.append(0.5 * (g + up(g, d)))
                div = sum(G[b][b] for b in range(D))
                tau = torch.stack([mu * (G[d][a] + G[a][d]) - (2.0 / 3.0 * mu * div if a == d else 0.0)
                                   for a in range(D)])
                en = (0.5 * (v + up(v, d)) * tau).sum(0) + kappa * (up(T, d) - T) / dx[d]
                F = F - torch.cat([torch.zeros_like(en)[None], tau, en[None]])
            out = out + (up(F, d, -1) - F) / dx[d]
        return out.reshape(-1)

    return f


def _f_ogrid(case, pb, nodes, device):
    """y -> f(y) on the O-grid: periodic in i, a wall below row 0, the far field above the last row."""
    x, y = (torch.as_tensor(a, device=device) for a in nodes)
    nx, ny = pb["n"]
    nxt = lambda a, k=1: torch.roll(a, -k, -1)  # noqa: E731
    X = torch.stack([x, y])
    p0, p1, p2, p3 = X[:, :-1], nxt(X)[:, :-1], nxt(X)[:, 1:], X[:, 1:]
    turn = lambda t: torch.stack([t[1], -t[0]])  # noqa: E731
    area = 0.5 * ((p2 - p0)[0] * (p3 - p1)[1] - (p3 - p1)[0] * (p2 - p0)[1])
    cen = 0.25 * (p0 + p1 + p2 + p3)
    Se = turn(p2 - p1)                                             # face i + 1/2
    Sn = torch.cat([turn(nxt(X)[:, :1] - X[:, :1]) * -1.0, turn(p3 - p2)], 1)   # faces j - 1/2, j = 0..ny
    de = nxt(cen) - cen
    dn = cen[:, 1:] - cen[:, :-1]
    dw = cen[:, 0] - 0.5 * (X[:, 0] + nxt(X)[:, 0])
    Uinf = torch.tensor(_freestream(), dtype=torch.float64, device=device)[:, None].expand(4, nx)
    t_wall, flux = 1.0, pb["flux"]

    def rotated(qL, qR, S):
        ln = torch.sqrt(S[0] ** 2 + S[1] ** 2)
        n = S / ln
        turned = lambda q: torch.stack([q[0], q[1] * n[0] + q[2] * n[1], q[2] * n[0] - q[1] * n[1], q[3]])  # noqa: E731
        F = _num_flux(flux, turned(qL), turned(qR), 0)
        return torch.stack([F[0], F[1] * n[0] - F[2] * n[1], F[1] * n[1] + F[2] * n[0], F[3]]) * ln

    def viscous(S, dc, across, along, uf, Tf, sign):
        # the gradient from the differences across and along the face: (across S + sign along (dc_y, -dc_x)) / (dc . S)
        J = (dc * S).sum(0)
        gx = (across * S[0] + sign * along * dc[1]) / J
        gy = (across * S[1] - sign * along * dc[0]) / J
        mu = MU_CYLINDER * Tf * torch.sqrt(Tf) * (1.0 + SUTHERLAND) / (Tf + SUTHERLAND)
        kap = mu * GAMMA / ((GAMMA - 1.0) * PRANDTL)
        div = gx[0] + gy[1]
        txx, tyy = (mu * (2 * g - 2.0 / 3.0 * div) for g in (gx[0], gy[1]))
        txy = mu * (gy[0] + gx[1])
        fx, fy = txx * S[0] + txy * S[1], txy * S[0] + tyy * S[1]
        return torch.stack([torch.zeros_like(fx), fx, fy, uf[0] * fx + uf[1] * fy + kap * (gx[2] * S[0] + gy[2] * S[1])])

    def f(z):
        q = _primitives(z.view(4, ny, nx))
        w = torch.cat([q[1:3], (q[3] / q[0])[None]])               # u, v, T
        mean = lambda a, b: 0.5 * (a + b)  # noqa: E731
        muscl = pb["recon"] == "muscl"
        si = _minmod(q - nxt(q, -1), nxt(q) - q) if muscl else torch.zeros_like(q)
        Fi = rotated(q + 0.5 * si, nxt(q - 0.5 * si), Se)
        gj = torch.cat([w[:, 1:2] - w[:, :1], 0.5 * (w[:, 2:] - w[:, :-2]), w[:, -1:] - w[:, -2:-1]], 1)
        Fi = Fi - viscous(Se, de, nxt(w) - w, mean(gj, nxt(gj)), mean(w, nxt(w)), mean(w, nxt(w))[2], -1.0)
        sj = torch.zeros_like(q)
        if muscl:
            sj = torch.cat([sj[:, :1], _minmod(q[:, 1:-1] - q[:, :-2], q[:, 2:] - q[:, 1:-1]), sj[:, -1:]], 1)
        Fj = rotated((q + 0.5 * sj)[:, :-1], (q - 0.5 * sj)[:, 1:], Sn[:, 1:-1])
        gi = 0.5 * (nxt(w) - nxt(w, -1))
        m = mean(w[:, :-1], w[:, 1:])
        Fj = Fj - viscous(Sn[:, 1:-1], dn, w[:, 1:] - w[:, :-1], mean(gi[:, :-1], gi[:, 1:]), m, m[2], 1.0)
        zero = torch.zeros_like(w[:, 0])
        wall = torch.stack([zero[0], q[3, 0] * Sn[0, 0], q[3, 0] * Sn[1, 0], zero[0]])
        across = torch.stack([w[0, 0], w[1, 0], w[2, 0] - t_wall])
        wall = wall - viscous(Sn[:, 0], dw, across, zero, zero, 0.5 * (w[2, 0] + t_wall), 1.0)
        far = rotated(q[:, -1], _primitives(Uinf), Sn[:, -1])
        Fj = torch.cat([wall[:, None], Fj, far[:, None]], 1)
        return ((nxt(Fi, -1) - Fi + Fj[:, :-1] - Fj[:, 1:]) / area).reshape(-1)

    return f


def _product(f, y, fy, fd):
    if fd:
        eps = math.sqrt((1.0 + float(y.norm())) * 2.0 ** -52)
        return lambda v, scale=1.0: (f(y + (eps / scale) * v) - fy) / (eps / scale)
    return lambda v, scale=1.0: torch.func.jvp(f, (y,), (v,))[1]


def _arnoldi(f, y, fy, M, fd):
    """Modified Gram-Schmidt: basis vectors and H, its entries by (row, column)."""
    V, H, J = [fy / fy.norm()], {}, _product(f, y, fy, fd)
    for j in range(M):
        w = J(V[j])
        for i in range(j + 1):
            H[i, j] = torch.dot(V[i], w)
            w = w - H[i, j] * V[i]
        if j + 1 < M:
            H[j + 1, j] = w.norm()
            V.append(w / H[j + 1, j])
    zero = torch.zeros_like(y[0])
    return V, torch.stack([torch.stack([H.get((i, j), zero) for j in range(M)]) for i in range(M)]) if M else None


def _step(f, y, h, tab, M, fd):
    F = f(y)
    A = V = H = None
    if M:
        V, H = _arnoldi(f, y, F, M, fd)
        A = torch.eye(M, dtype=y.dtype, device=y.device) - h * tab["gamma"] * H
    ks, lams = [], []
    for i in range(tab["s"]):
        if i:
            Y = y
            for j in range(i):
                if tab["alpha"][i][j]:
                    Y = Y + tab["alpha"][i][j] * ks[j]
            F = f(Y)
        if not M:
            ks.append(h * F)
            continue
        phi = torch.stack([torch.dot(v, F) for v in V])
        g = torch.zeros_like(phi)
        for j in range(i):
            g = g + tab["gam"][i][j] * lams[j]
        lams.append(torch.linalg.solve(A, h * phi + h * (H @ g)))
        k = h * F
        for c in range(M):
            k = k + (lams[i][c] - h * phi[c]) * V[c]
        ks.append(k)
    for b, k in zip(tab["b"], ks):
        y = y + b * k
    return y


def _adaptive(f, y, case, h, tab):
    t, T, H, tol, calm, counts = 0.0, case["steps"] * h, h, case["tol"], True, [0, 0]
    while t < T and sum(counts) < 200:
        last = t + H >= T
        H = T - t if last else H
        full = _step(f, y, H, tab, case["M"], True)
        half = _step(f, _step(f, y, 0.5 * H, tab, case["M"], True), 0.5 * H, tab, case["M"], True)
        e = (half - full) / (15.0 * (tol + tol * torch.maximum(y.abs(), half.abs())))
        err = math.sqrt(float((e * e).mean()))
        ok = err <= 1.0
        counts[0 if ok else 1] += 1
        if ok:
            t, y = (T if last else t + H), half
        most = 4.0 if ok and calm else 1.0
        H *= (min(most, max(0.2, 0.9 * err ** -0.2)) if err > 0 else most) if math.isfinite(err) else 0.2
        calm = ok
    return {"y": y, "accepted": counts[0], "rejected": counts[1]}


def exact(case, seed):
    if case["call"] == "eigs":   # the dense spectrum of 32768 unknowns takes minutes
        return None
    device = "cuda" if torch.cuda.is_available() else "cpu"
    pb, nodes, y, v, w, h = _inputs(case, seed, device)
    f = _f_ogrid(case, pb, nodes, device) if nodes is not None else _f_box(case, pb)
    tab, M = ri.rok4_tableau(), case["M"]
    if case["call"] == "gradient":
        states = [y]
        with torch.no_grad():
            for _ in range(case["steps"]):
                states.append(_step(f, states[-1], h, tab, M, False))
        last = states[-1].requires_grad_(True)
        (g,) = torch.autograd.grad(_kinetic_energy(last), last)
        for yn in reversed(states[:-1]):
            yn = yn.detach().requires_grad_(True)
            (g,) = torch.autograd.grad(_step(f, yn, h, tab, M, False), yn, g)
        return {"y": last.detach(), "gradient": g}
    if case["call"] == "operators":
        z = y.clone().requires_grad_(True)
        (jtw,) = torch.autograd.grad(f(z), z, w)
        with torch.no_grad():
            F = f(y)
            return {"f": F, "jv_fd": _product(f, y, F, True)(v, float(v.norm())),
                    "jv": _product(f, y, F, False)(v), "jtw": jtw}
    with torch.no_grad():
        if case["call"] == "step":
            return _step(f, y, h, tab, M, case["jvp"] == "fd")
        if case["call"] == "adaptive":
            return _adaptive(f, y, case, h, tab)
        V, H = _arnoldi(f, y, f(y), M, False)
        return {"V": torch.stack(V), "H": H, "m": M}
