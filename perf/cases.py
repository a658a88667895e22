"""The work that a program using this framework has it do, as measurable cases.

A case is a dict of plain values.  "do" names the call sequence:

* recover    es_con2prim and es_cfl on a stored state (what a restart or an output step does)
* setup      es_metrics with the initial Jacobian and es_prim2con (the start of every simulation)
* residual   es_residual on a moving curvilinear mesh (the hot call of a method-of-lines driver)
* step       es_rk3_step: one whole adaptive or static SSP-RK3 step, in place
* moving     es_rk3_step_moving: one step on a prescribed moving mesh with a given time step
* adjoint    autograd.rk3_step and its gradient (checkpointed step, then the step's VJP)

and "flow" the initial data: the advected sine, four constant quadrants, the 3D blast, the RMHD
vortex, and a smooth seeded state in which every field varies (gradients are taken there: where a
field is constant to rounding, rounding decides the sign switch of its dissipation, and with it the
gradient).

exact() evaluates the same method in plain torch in 64 bits: conservative metrics, two-point
entropy conservative fluxes, WENO dissipation on scaled entropy variables, the Godunov-Powell
source, con2prim by Newton, mesh redistribution and Shu-Osher stages; gradients by torch's own
reverse mode with the mesh, the time step and the switches held (RMHD: the face eigen-structure
too).  Large magnetised fields have no exact value: it solves one eigenproblem per face.
"""
from __future__ import annotations

import math

import torch

from paper_2107_12027_amd import autograd, es, workloads as wl

GAMMA = 5.0 / 3.0


def _case(name, do, phys, n, bc, flow, p=3, dissipation=1, mixed=0, form=-1, sigma=0, alpha=0.0, sweeps=10,
          cfl=0.4):
    """n: nodes along xi_1, xi_2(, xi_3); bc: one letter per axis, p(eriodic) or o(utflow); form -1: static mesh."""
    c = {"name": name, "do": do, "phys": phys, "dim": len(n), "bc": bc, "flow": flow, "p": p,
         "dissipation": dissipation, "mixed": mixed, "form": form, "sigma": sigma, "alpha": alpha, "sweeps": sweeps,
         "cfl": cfl}
    for k in range(3):
        c["n%d" % k] = int(n[k]) if k < len(n) else 1
    return c


def listed():
    return [
        # the smallest call: the primitive state and the time step of a small stored field
        _case("recover_33x47", "recover", "rhd", (33, 47), "po", "quadrants"),
        # the advected sine of the accuracy tests: a whole adaptive step where latency and launches count
        _case("step_sine_64", "step", "rhd", (64, 64), "pp", "sine", form=1, alpha=10.0),
        # a 2D Riemann problem at the usual production size: ordinary adaptive steps
        _case("step_quadrants_400", "step", "rhd", (400, 400), "oo", "quadrants", form=0, sigma=1, alpha=1200.0),
        # the 3D blast that the benchmark quotes: the largest step
        _case("step_blast_128", "step", "rhd", (128, 128, 128), "ooo", "blast", form=0, alpha=800.0, sweeps=5,
              cfl=0.3),
        # the residual alone, ragged 3D box with mixed boundaries
        _case("residual_131x67x45", "residual", "rhd", (131, 67, 45), "pop", "smooth"),
        # the FP32-mixed form of the residual
        _case("residual_mixed_96x80x72", "residual", "rhd", (96, 80, 72), "ooo", "smooth", mixed=1),
        # the eighth-order scheme in 2D
        _case("residual_p4_301x257", "residual", "rhd", (301, 257), "oo", "smooth", p=4),
        # what every 3D simulation does before its first step
        _case("setup_128", "setup", "rhd", (128, 128, 128), "ooo", "smooth"),
        # a magnetised flow at the size of the rotor runs, adaptive as the RMHD examples are
        _case("step_magnetised_512", "step", "rmhd", (512, 512), "oo", "smooth", form=0, sigma=1, alpha=200.0),
        # the entropy conservative accuracy runs on a prescribed mesh (thousands of small steps)
        _case("moving_vortex_160", "moving", "rmhd", (160, 160), "pp", "vortex", dissipation=0),
        # gradient studies: a magnetised flow on a static 2D mesh, and a 3D flow on its adaptive mesh
        _case("adjoint_magnetised_256", "adjoint", "rmhd", (256, 256), "pp", "smooth"),
        _case("adjoint_72x64x56", "adjoint", "rhd", (72, 64, 56), "ooo", "smooth", form=0, alpha=200.0, sweeps=5,
              cfl=0.3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["recover", "setup", "residual", "residual", "residual", "step", "step", "step", "moving", "adjoint"])
    phys = "rmhd" if do == "moving" else rng.choice(["rhd", "rhd", "rmhd"])
    dim = 2 if do == "moving" else rng.choice([2, 3])
    magnetised = phys == "rmhd"
    # most nodes of one call: the cost of a magnetised or differentiated node is far higher
    most = {"recover": 2_000_000, "setup": 2_000_000, "residual": 1_200_000, "step": 900_000, "moving": 90_000,
            "adjoint": 250_000}[do]
    if magnetised and do in ("residual", "step", "adjoint"):
        most //= 8 if do != "adjoint" else 4
    nodes = _log_int(rng, 1_500, most)
    side = nodes ** (1.0 / dim)
    n = [max(11, int(side * rng.uniform(0.6, 1.5))) for _ in range(dim)]
    bc = "pp" if do == "moving" else "".join(rng.choice("po") for _ in range(dim))
    p = rng.choice([3, 3, 2] if do == "adjoint" else [3, 3, 3, 2, 4])
    mixed = int(do == "residual" and not magnetised and rng.random() < 0.25)
    adaptive = do in ("step", "adjoint") and rng.random() < 0.7
    form = rng.choice([0, 1, 2]) if adaptive else -1
    return _case("", do, phys, n, bc, "vortex" if do == "moving" else "smooth", p=p,
                 dissipation=0 if do == "moving" else 1, mixed=mixed, form=form, sigma=rng.choice([0, 1]),
                 alpha={0: 200.0, 1: 10.0, 2: 20.0, -1: 0.0}[form], sweeps=rng.choice([5, 10]),
                 cfl=0.4 if dim == 2 else 0.3)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

class _Box:
    """The computational box of a case: sizes, spacings, boundaries and the physical domain."""

    def __init__(self, case):
        self.dim = case["dim"]
        self.n = tuple(case["n%d" % k] for k in range(self.dim))
        self.periodic = tuple(b == "p" for b in case["bc"])
        vortex = case["flow"] == "vortex"
        self.lo, self.length = (-wl.VORTEX_R, 2.0 * wl.VORTEX_R) if vortex else (0.0, 1.0)
        self.h = tuple(1.0 / n if per else 1.0 / (n - 1) for n, per in zip(self.n, self.periodic))
        self.shape = tuple(reversed(self.n))
        self.p = case["p"]
        self.ng = max(3, case["p"])
        self.rmhd = case["phys"] == "rmhd"
        # conservative and primitive slots of (rho, u, p, B) that the system keeps
        self.slots = list(range(8)) if self.rmhd else ([0, 1, 2, 4] if self.dim == 2 else [0, 1, 2, 3, 4])

    def xi(self):
        """Computational coordinates of the nodes, (dim, *shape)."""
        axes = [torch.arange(n, dtype=torch.float64, device="cuda") * h for n, h in zip(self.n, self.h)]
        grids = torch.meshgrid(*reversed(axes), indexing="ij")
        return torch.stack(list(reversed(grids)))


def _modes(gen, xi, count=4):
    """A seeded sum of Fourier modes of xi with values in about [-1, 1]."""
    f = torch.zeros_like(xi[0])
    for _ in range(count):
        k = torch.randint(-2, 3, (xi.shape[0],), generator=gen).tolist()
        if not any(k):
            k[0] = 1
        phase = 2 * math.pi * torch.rand(1, generator=gen).item()
        f = f + torch.sin(2 * math.pi * sum(a * x for a, x in zip(k, xi)) + phase) / count
    return f


def _inputs(case, seed):
    """(box, P, x, xdot): the primitive state (rho, u, p, B) (8, *shape), mesh and mesh velocity."""
    b = _Box(case)
    gen = torch.Generator().manual_seed(int(seed))
    rand = lambda: torch.rand(1, generator=gen).item()  # noqa: E731
    xi = b.xi()
    x = b.lo + b.length * xi
    xdot = torch.zeros_like(x)
    v = torch.zeros((3,) + b.shape, dtype=torch.float64, device="cuda")
    B = torch.zeros_like(v)
    rho, p = torch.ones_like(xi[0]), torch.ones_like(xi[0])
    flow = case["flow"]
    if case["do"] in ("residual", "setup"):
        # a smooth curvilinear mesh in motion, its bounded edges kept in place
        for k in range(b.dim):
            fixed = 1.0 if b.periodic[k] else torch.sin(math.pi * xi[k])
            x[k] += 0.03 * b.length * fixed * _modes(gen, xi)
            xdot[k] += 0.1 * b.length * fixed * _modes(gen, xi)
    if flow == "sine":
        rho = 1.0 + 0.2 * torch.sin(2 * math.pi * (xi[0] + xi[1] + rand()))
        v[0] += 0.2
        v[1] += 0.2
    elif flow == "quadrants":
        # Riemann problem II: (rho, v1, v2, p) in the four quadrants, each state moved by up to 2 %
        east, north = xi[0] > 0.5, xi[1] > 0.5
        for sel, (r, v1, v2, pr) in zip((east & north, ~east & north, ~east & ~north, east & ~north),
                                        wl.RIEMANN_2D[2]):
            rho[sel] = r * (0.98 + 0.04 * rand())
            p[sel] = pr * (0.98 + 0.04 * rand())
            v[0][sel] = v1
            v[1][sel] = v2
    elif flow == "blast":
        noise = torch.rand(b.shape, generator=gen, dtype=torch.float64).cuda()
        rho = 0.99 + 0.02 * noise
        p = torch.where(sum((c - 0.5) ** 2 for c in xi) < 0.01, 1000.0, 1.0).to(torch.float64)
    elif flow == "vortex":
        t = 4.0 * rand()
        amp = wl.vortex_mesh_amplitude
        s = torch.stack([torch.sin(3 * math.pi * x[1 - k] / wl.VORTEX_R) for k in range(2)])
        dt = _vortex_dt(b)
        xdot = (amp(t + dt) - amp(t)) / dt * s
        x = x + amp(t) * s
        state = wl.vortex2d_state(x[0].cpu().numpy(), x[1].cpu().numpy(), t)
        rho, v, p, B = (torch.from_numpy(a).cuda() for a in state)
    else:
        rho = 1.0 + 0.2 * _modes(gen, xi)
        p = 1.0 + 0.2 * _modes(gen, xi)
        kept = 3 if b.rmhd or b.dim == 3 else 2
        for c in range(kept):
            v[c] = 0.1 * (c + 1) + 0.15 * _modes(gen, xi)
        if b.rmhd:
            for c, level in enumerate((0.6, 0.45, 0.35)):
                B[c] = level + 0.1 * _modes(gen, xi)
    u = v / torch.sqrt(1.0 - (v * v).sum(0))
    return b, torch.cat([rho[None], u, p[None], B]).contiguous(), x.contiguous(), xdot.contiguous()


def _vortex_dt(b):
    return 0.4 * b.h[0] ** 2


def _adjoint_dt(b):
    return 0.1 * min(b.h)


def _cotangents(b, seed):
    """Seeded cotangents of (U, J) after the step."""
    gen = torch.Generator().manual_seed(int(seed) + 1)
    xi = b.xi()
    return torch.stack([_modes(gen, xi) for _ in b.slots]), _modes(gen, xi)


class _State:
    pass


def prepare(case, seed):
    b, P, x, xdot = _inputs(case, seed)
    full = lambda t, fill: tuple(t[k] if k < b.dim else fill for k in range(3))  # noqa: E731
    per = full(b.periodic, True)
    grid = wl.Grid(b.dim, full(b.n, 1), tuple(wl.PERIODIC if q else wl.OUTFLOW for q in per), full(b.h, 1.0),
                   tuple(b.length if k < b.dim and per[k] else 0.0 for k in range(3)), (b.lo,) * 3, (b.length,) * 3)
    s = _State()
    s.case = case
    s.ctx = ctx = es.Context(
        grid, wl.Scheme(phys=wl.RMHD if b.rmhd else wl.RHD, gamma=GAMMA, order_p=case["p"],
                        dissipation=case["dissipation"], cfl=case["cfl"], mixed=case["mixed"]),
        wl.Monitor(enabled=int(case["form"] >= 0), sigma=case["sigma"], form=max(0, case["form"]),
                   alpha=case["alpha"], alpha2=0.5 * case["alpha"], sweeps=case["sweeps"]))
    new = lambda *shape: torch.empty(shape, dtype=torch.float64, device="cuda")  # noqa: E731
    shape, padded = ctx.shape(), ctx.padded_shape()
    s.x, s.xdot, s.prim0 = x, xdot, P[b.slots].contiguous()
    s.met, s.J, s.U, s.dt = new(ctx.nmet, *padded), new(*shape), new(ctx.m, *shape), new(1)
    if case["do"] == "setup":
        return s
    ctx.metrics(x, None, s.met, s.J)
    ctx.prim2con(s.prim0, s.J, s.U)
    if case["do"] in ("recover", "residual"):
        s.prim = new(ctx.nprim, *padded)
    if case["do"] == "residual":
        ctx.con2prim(s.U, s.J, s.prim)
        ctx.metrics(x, xdot, s.met)
        s.dU, s.dJ = new(ctx.m, *shape), new(*shape)
    elif case["do"] == "moving":
        s.fixed_dt = torch.full((1,), _vortex_dt(b), dtype=torch.float64, device="cuda")
    elif case["do"] == "adjoint":
        s.lam = _cotangents(b, seed)
        s.fixed_dt = None if case["form"] >= 0 else torch.full((1,), _adjoint_dt(b), dtype=torch.float64,
                                                               device="cuda")
    return s


def run(s):
    do, ctx = s.case["do"], s.ctx
    if do == "recover":
        ctx.con2prim(s.U, s.J, s.prim)
        ctx.cfl(s.prim, s.met, s.J, s.dt)
        return s.prim, s.dt
    if do == "setup":
        ctx.metrics(s.x, None, s.met, s.J)
        ctx.prim2con(s.prim0, s.J, s.U)
        return s.met, s.J, s.U
    if do == "residual":
        ctx.residual(s.prim, s.met, s.dU, s.dJ)
        return s.dU, s.dJ
    if do == "step":
        ctx.rk3_step(s.U, s.J, s.x, s.xdot, s.dt)
        return s.U, s.J, s.x, s.xdot, s.dt
    if do == "moving":
        ctx.rk3_step_moving(s.U, s.J, s.x, s.xdot, s.dt, s.fixed_dt)
        return s.U, s.J, s.x
    U, J = s.U.detach().requires_grad_(), s.J.detach().requires_grad_()
    U1, J1, x1, dt = autograd.rk3_step(U, J, ctx, s.x, s.fixed_dt)
    gU, gJ = torch.autograd.grad((U1, J1), (U, J), s.lam)
    return U1.detach(), J1.detach(), x1, dt, gU, gJ


def work(case):
    """Fields read and written once; operations of the pair fluxes (about 100, RMHD 250, per pair), of one face's
    dissipation (600; the eigen-structure of an RMHD face 6000) and of the per-node maps, whatever the code does."""
    b = _Box(case)
    d, m = b.dim, len(b.slots)
    nodes = math.prod(b.n)
    padded = math.prod(n + 2 * b.ng for n in b.n)
    nmet = d * (d + 1)
    pair = (250 if b.rmhd else 100) * case["p"]
    face = (6000 if b.rmhd else 600) if case["dissipation"] else 0
    residual = d * (pair + face)
    node = 200
    do = case["do"]
    if do == "recover":
        return {"bytes": 8 * (nodes * (m + 1) + padded * (m + 2 + nmet)), "flops": nodes * 2 * node}
    if do == "setup":
        return {"bytes": 8 * (nodes * (d + 2 * m + 1) + padded * nmet), "flops": nodes * (node + 60 * d)}
    if do == "residual":
        return {"bytes": 8 * (padded * (m + 2 + nmet) + nodes * (m + 1)), "flops": nodes * residual}
    mesh = 30 * (case["sweeps"] + 3) if case["form"] >= 0 else 0
    step = 3 * (residual + node) + mesh
    state = 8 * nodes * (m + 1 + d)
    if do == "adjoint":
        return {"bytes": 2 * state + 8 * nodes * (4 * (m + 1) + 3 * (m + 1) + 2 * d), "flops": nodes * 4 * step}
    return {"bytes": 2 * state + 8 * nodes * d, "flops": nodes * step}


# ---------------------------------------------------------------------------
# the same method in plain torch, 64 bits
# ---------------------------------------------------------------------------

def _axis(t, k):
    return t.ndim - 1 - k


def _cut(t, k, lo, count):
    return t.narrow(_axis(t, k), lo, count)


def _crop(t, k, w):
    return _cut(t, k, w, t.shape[_axis(t, k)] - 2 * w)


def _extend(b, f, w, rule, comp=-1):
    """A node field continued by w layers on every axis: "solution" (wrap / edge copy), "mesh" (wrap with the
    period added to coordinate comp / odd reflection) or "velocity" (wrap / odd reflection)."""
    for k in range(b.dim):
        ax, n = _axis(f, k), b.n[k]
        i = torch.arange(-w, n + w, device=f.device)
        if b.periodic[k]:
            g = f.index_select(ax, i % n)
            if rule == "mesh" and comp == k:
                turn = torch.div(i, n, rounding_mode="floor").to(f.dtype) * b.length
                g = g + turn.reshape([-1 if a == ax else 1 for a in range(f.ndim)])
        else:
            g = f.index_select(ax, i.clamp(0, n - 1))
            if rule != "solution":
                mirror = f.index_select(ax, torch.where(i < 0, -i, torch.where(i >= n, 2 * (n - 1) - i, i)))
                outside = ((i < 0) | (i >= n)).reshape([-1 if a == ax else 1 for a in range(f.ndim)])
                g = torch.where(outside, 2.0 * g - mirror, g)
        f = g
    return f


_ALPHA = {2: (4 / 3, -1 / 6), 3: (3 / 2, -3 / 10, 1 / 30), 4: (8 / 5, -2 / 5, 8 / 105, -1 / 140)}


def _diff(f, k, p):
    """Central difference of order 2p along axis k; p layers are lost on either side."""
    n = f.shape[_axis(f, k)] - 2 * p
    return sum(0.5 * a * (_cut(f, k, p + m, n) - _cut(f, k, p - m, n)) for m, a in enumerate(_ALPHA[p], 1))


def _metrics(b, x, xdot=None):
    """met[k] = (J dxi_k/dt, J dxi_k/dx_1, ..) on the padded box."""
    p, ng, d = b.p, b.ng, b.dim
    X = [_extend(b, x[c], 2 * ng, "mesh", c) for c in range(d)]

    def to_padded(f, lost):
        for k in range(d):
            f = _crop(f, k, ng - lost.count(k) * p)
        return f

    S = []
    for k in range(d):
        if d == 2:
            o = 1 - k
            sign = 1.0 if k == 0 else -1.0
            S.append([sign * to_padded(_diff(X[1], o, p), [o]) / b.h[o],
                      -sign * to_padded(_diff(X[0], o, p), [o]) / b.h[o]])
            continue
        k1, k2 = (k + 1) % 3, (k + 2) % 3
        row = []
        for j in range(3):
            a, c = X[(j + 1) % 3], X[(j + 2) % 3]
            first = _diff(_diff(a, k1, p) * _crop(c, k1, p), k2, p)
            second = _diff(_diff(a, k2, p) * _crop(c, k2, p), k1, p)
            row.append(to_padded(first - second, [k1, k2]) / (b.h[k1] * b.h[k2]))
        S.append(row)
    V = None if xdot is None else [_extend(b, xdot[c], ng, "velocity") for c in range(d)]
    return [torch.stack([torch.zeros_like(r[0]) if V is None else -sum(v * s for v, s in zip(V, r))] + r) for r in S]


def _inner(b, f):
    for k in range(b.dim):
        f = _crop(f, k, b.ng)
    return f


def _jacobian(b, x):
    p, d = b.p, b.dim
    D = []       # D[k][c] = delta_k x_c / h_k on the interior
    for k in range(d):
        row = []
        for c in range(d if d == 2 else 1):
            f = _diff(_extend(b, x[c], p, "mesh", c), k, p) / b.h[k]
            for o in range(d):
                f = f if o == k else _crop(f, o, p)
            row.append(f)
        D.append(row)
    if d == 2:
        return D[0][0] * D[1][1] - D[1][0] * D[0][1]
    return sum(_inner(b, m[1]) * row[0] for m, row in zip(_metrics(b, x), D))


def _thermo(P):
    """W, v, b^0, b, |b|^2 of (rho, u, p, B)."""
    u, B = P[1:4], P[5:8]
    W = torch.sqrt(1.0 + (u * u).sum(0))
    b0 = (u * B).sum(0)
    bv = (B + b0 * u) / W
    return W, u / W, b0, bv, (bv * bv).sum(0) - b0 * b0


def _conserved(P):
    W, v, b0, bv, b2 = _thermo(P)
    B = P[5:8]
    Z = (P[0] + GAMMA / (GAMMA - 1) * P[4]) * W * W
    B2 = (B * B).sum(0)
    m = (Z + B2) * v - b0 / W * B
    return torch.cat([(P[0] * W)[None], m, (Z - P[4] - 0.5 * b2 + B2)[None], B])


def _flux_x(P):
    W, v, b0, bv, b2 = _thermo(P)
    B = P[5:8]
    U = _conserved(P)
    m = U[1:4] * v[0] - B[0] * bv / W
    m = torch.cat([(m[0] + P[4] + 0.5 * b2)[None], m[1:]])
    return torch.cat([(U[0] * v[0])[None], m, U[1][None], v[0] * B - B[0] * v])


def _phi_prime(P):
    W, v, b0, bv, _ = _thermo(P)
    return torch.cat([torch.zeros_like(W)[None], bv / W, (b0 / W)[None], v])


def _entropy(P):
    W, _, _, bv, _ = _thermo(P)
    beta = P[0] / P[4]
    first = GAMMA / (GAMMA - 1) + torch.log(P[0]) + torch.log(beta) / (GAMMA - 1) + beta
    return torch.cat([first[None], beta * P[1:4], (-beta * W)[None], beta * bv])


def _from_entropy(V):
    beta = torch.sqrt(V[4] ** 2 - (V[1:4] ** 2).sum(0))
    u, bv, W = V[1:4] / beta, V[5:8] / beta, -V[4] / beta
    rho = torch.exp(V[0] - GAMMA / (GAMMA - 1) - torch.log(beta) / (GAMMA - 1) - beta)
    b0 = (u * bv).sum(0) / W
    return torch.cat([rho[None], u, (rho / beta)[None], W * bv - b0 * u])


def _full(b, U):
    """The kept conservative slots in all eight."""
    out = list(torch.zeros_like(U[:1]).expand(8, *U.shape[1:]))
    for i, c in enumerate(b.slots):
        out[c] = U[i]
    return torch.stack(out)


def _recover(b, Uc, J):
    """(rho, u, p, B) of Ucurv / J: bisection and Newton on the scalar equation in Z = rho h W^2; the last Newton
    step carries the derivative (the implicit function rule)."""
    U = _full(b, Uc) / J
    D, m, E, B = U[0], U[1:4], U[4], U[5:8]
    gm = (GAMMA - 1) / GAMMA

    def f(Z, D, m, E, B):
        mB, B2, m2 = (m * B).sum(0), (B * B).sum(0), (m * m).sum(0)
        v2 = (Z * Z * m2 + mB * mB * (2 * Z + B2)) / (Z * Z * (Z + B2) ** 2)
        iW2 = 1.0 - v2
        iW = torch.sqrt(iW2.clamp(min=1e-300))
        g = Z - gm * (Z * iW2 - D * iW) + B2 - 0.5 * B2 * iW2 - 0.5 * mB * mB / (Z * Z) - E
        return torch.where(iW2 > 0, g, -1.0), v2

    with torch.no_grad():
        args = [t.detach() for t in (D, m, E, B)]
        lo = torch.zeros_like(E)
        hi = 2.0 * (E.detach() + 1.0) + (B.detach() ** 2).sum(0)
        for _ in range(60):
            Z = 0.5 * (lo + hi)
            low = f(Z, *args)[0] < 0
            lo, hi = torch.where(low, Z, lo), torch.where(low, hi, Z)
        Z = 0.5 * (lo + hi)
    with torch.enable_grad():
        z = Z.detach().requires_grad_()
        slope = torch.autograd.grad(f(z, *args)[0].sum(), z)[0]
    Z = Z - f(Z, D, m, E, B)[0] / slope
    mB, B2 = (m * B).sum(0), (B * B).sum(0)
    v = (m + mB / Z * B) / (Z + B2)
    iW = torch.sqrt(1.0 - (v * v).sum(0))
    rho = D * iW
    return torch.cat([rho[None], v / iW, (gm * (Z * iW * iW - rho))[None], B])


def _log_mean(a, b):
    f = (a - b) / (a + b)
    small = f.abs() < 0.1
    g = torch.where(small, f, torch.zeros_like(f))
    series = sum(g ** (2 * k) / (2 * k + 1) for k in range(9))
    g = torch.where(small, torch.full_like(f, 0.5), f)
    return 0.5 * (a + b) / torch.where(small, series, torch.atanh(g) / g)


def _pair(b, Pl, Pr, al, ar):
    """Two-point entropy conservative flux (8 slots), VCL value and source pair between two states."""
    mean = lambda f: 0.5 * (f(Pl) + f(Pr))  # noqa: E731
    Wl, _, b0l, bl, _ = _thermo(Pl)
    Wr, _, b0r, br, _ = _thermo(Pr)
    av = lambda x, y: 0.5 * (x + y)  # noqa: E731
    rho_ln = _log_mean(Pl[0], Pr[0])
    a0 = 1.0 + 1.0 / ((GAMMA - 1) * _log_mean(Pl[0] / Pl[4], Pr[0] / Pr[4]))
    rho, beta = mean(lambda P: P[0]), mean(lambda P: P[0] / P[4])
    u, B, W, b0, bb = av(Pl[1:4], Pr[1:4]), av(Pl[5:8], Pr[5:8]), av(Wl, Wr), av(b0l, b0r), av(bl, br)
    Wb0, Wb02 = av(Wl * b0l, Wr * b0r), av(Wl * b0l ** 2, Wr * b0r ** 2)
    Wbk2 = av(Wl * bl ** 2, Wr * br ** 2)
    sl, sr = (bl ** 2).sum(0), (br ** 2).sum(0)
    s, b02 = av(sl, sr), av(b0l ** 2, b0r ** 2)
    us, ub02 = av(Pl[1:4] * sl, Pr[1:4] * sr), av(Pl[1:4] * b0l ** 2, Pr[1:4] * b0r ** 2)
    gap = W * W - (u * u).sum(0)
    # the part along the time metric
    UB = W * bb - Wb0 * u / W
    R1 = -a0 * rho_ln * W - 0.5 * Wb02 + (0.5 * Wbk2 - bb * UB).sum(0)
    Rk = ((rho + 0.5 * beta * s + 0.5 * beta * Wb02 / W) * u - beta * Wb0 * bb) / W
    U5 = ((u * Rk).sum(0) / beta - R1) * W / gap
    at = 0.5 * (al[0] + ar[0])
    F = at * torch.cat([(rho_ln * W)[None], u * U5 / W + Rk / beta, U5[None], UB])
    bt = 0.0
    for j in range(b.dim):
        c0 = u[j] * b0 + B[j]
        FB = u[j] * bb - c0 * u / W
        Pk = -c0 * beta / W * (bb - b0 * u / W)
        push = rho + 0.5 * beta * (s - b02)
        Pk = torch.stack([Pk[i] + push if i == j else Pk[i] for i in range(3)])
        Q = 0.5 * (us[j] - ub02[j]) - B[j] * b0
        F5 = W * (a0 * rho_ln * u[j] + (u * Pk).sum(0) / beta + (bb * FB).sum(0) - Q) / gap
        aj = 0.5 * (al[1 + j] + ar[1 + j])
        F = F + aj * torch.cat([(rho_ln * u[j])[None], u * F5 / W + Pk / beta, F5[None], FB])
        bt = bt + aj * B[j]
    return F, at, bt


def _weno(v, eps=1e-6):
    """WENO-JS value at the right of the middle node from 2p - 1 point values."""
    if len(v) == 3:
        a, b, c = v
        q = [(3 * b - a) / 2, (b + c) / 2]
        beta = [(b - a) ** 2, (c - b) ** 2]
        lin = [1 / 3, 2 / 3]
    elif len(v) == 5:
        a, b, c, d, e = v
        q = [(2 * a - 7 * b + 11 * c) / 6, (-b + 5 * c + 2 * d) / 6, (2 * c + 5 * d - e) / 6]
        beta = [13 / 12 * (a - 2 * b + c) ** 2 + (a - 4 * b + 3 * c) ** 2 / 4,
                13 / 12 * (b - 2 * c + d) ** 2 + (b - d) ** 2 / 4,
                13 / 12 * (c - 2 * d + e) ** 2 + (3 * c - 4 * d + e) ** 2 / 4]
        lin = [0.1, 0.6, 0.3]
    else:
        q, beta = [], []
        lin = [1 / 35, 12 / 35, 18 / 35, 4 / 35]
        value = ((-3, 13, -23, 25), (1, -5, 13, 3), (-1, 7, 7, -1), (3, 13, -5, 1))
        first = ((-2, 9, -18, 11), (1, -6, 3, 2), (-2, -3, 6, -1), (-11, 18, -9, 2))
        second = ((-1, 4, -5, 2), (0, 1, -2, 1), (1, -2, 1, 0), (2, -5, 4, -1))
        dot = lambda c, w: sum(x * y for x, y in zip(c, w))  # noqa: E731
        for k in range(4):
            w = v[k:k + 4]
            q.append(dot(value[k], w) / 12)
            beta.append(dot(first[k], w) ** 2 / 36 + 13 / 12 * dot(second[k], w) ** 2
                        + 781 / 720 * dot((-1, 3, -3, 1), w) ** 2)
    wt = [g / (eps + s) ** 2 for g, s in zip(lin, beta)]
    return sum(w * x for w, x in zip(wt, q)) / sum(wt)


def _frame(n):
    """Rotation with first row n (3, N): rows n, (-n2, n1, 0)/r, (-n3 n1/r, -n3 n2/r, r)."""
    r = torch.sqrt(n[0] ** 2 + n[1] ** 2)
    flat = r > 0
    s = torch.where(flat, r, torch.ones_like(r))
    z, one = torch.zeros_like(r), torch.ones_like(r)
    row2 = torch.stack([torch.where(flat, -n[1] / s, z), torch.where(flat, n[0] / s, one), z])
    row3 = torch.stack([torch.where(flat, -n[2] * n[0] / s, -n[2]), -n[2] * n[1] / s, r])
    return torch.stack([n, row2, row3])


def _turn(T, A, back=False):
    spec = "ji...,j...->i..." if back else "ij...,j...->i..."
    return torch.cat([A[:1], torch.einsum(spec, T, A[1:4]), A[4:5], torch.einsum(spec, T, A[5:8])])


def _eigen_rhd(b, Vm):
    """Characteristic speeds (m, ..) and scaled right eigenvectors [column][8 slots] at the rotated mean entropy
    variables: the acoustic pair, then the basis of the v_n cluster seeded by D and the transverse momenta."""
    beta = torch.sqrt(Vm[4] ** 2 - (Vm[1:4] ** 2).sum(0))
    W, v = -Vm[4] / beta, -Vm[1:4] / Vm[4]
    rho = torch.exp(Vm[0] - GAMMA / (GAMMA - 1) - torch.log(beta) / (GAMMA - 1) - beta)
    p, h = rho / beta, 1.0 + GAMMA / (GAMMA - 1) / beta
    c2 = GAMMA / (beta * h)
    v2, vn = (v * v).sum(0), v[0]
    root = torch.sqrt((1 - v2) * (1 - v2 * c2 - vn * vn * (1 - c2)) * c2)
    z = torch.zeros_like(W)
    cols, lam = [], []
    for sign in (-1.0, 1.0):
        la = (vn * (1 - c2) + sign * root) / (1 - v2 * c2)
        A = h * W * (1 - vn * vn) / (1 - vn * la)
        f = torch.sqrt(0.5 * p / h * (W * (1 / c2 - 1) + la / (W * (la - vn))))
        cols.append(f * torch.stack([z + 1, A * la, h * W * v[1], h * W * v[2], A, z, z, z]))
        lam.append(la)
    cols.append(torch.sqrt(rho * W * (GAMMA - 1) / GAMMA)
                * torch.stack([z + 1, W * v[0], W * v[1], W * v[2], W, z, z, z]))
    shear = lambda s, w, e1, e2: s * torch.stack([  # noqa: E731
        W * w, 2 * h * W * W * w * v[0], h * (2 * W * W * w * v[1] + e1), h * (2 * W * W * w * v[2] + e2),
        2 * h * W * W * w, z, z, z])
    g1 = 1 + W * W * v[1] ** 2
    cols.append(shear(torch.sqrt(p * W / (h * g1)), v[1], z + 1, z))
    lam += [vn, vn]
    if b.dim == 3:
        k = W * W * v[1] * v[2] / g1
        gt = 1 + W * W * (v[1] ** 2 + v[2] ** 2)
        cols.append(shear(torch.sqrt(p * W * g1 / (h * gt)), v[2] - k * v[1], -k, z + 1))
        lam.append(vn)
    return torch.stack(lam), torch.stack(cols)


def _eigen_rmhd(Vm):
    """As _eigen_rhd from the symmetric pencil (dF/dV, dU/dV) with complex-step Jacobians; states whose only close
    eigenvalues are the v_n pair, which takes the basis seeded by D and B_n.  No derivative is taken."""
    P = _from_entropy(Vm.detach())
    shape = P.shape[1:]
    P = P.reshape(8, -1)
    step = 1e-30
    Z = P[:, None].expand(8, 8, -1) + 1j * step * torch.eye(8, dtype=torch.float64, device=P.device)[:, :, None]
    jac = lambda f: (f(Z).imag / step).permute(2, 0, 1)  # noqa: E731
    JU, JF, JV = jac(_conserved), jac(_flux_x), jac(_entropy)
    JF[:, :, 5] += _phi_prime(P).T
    inv = torch.linalg.inv(JV)
    A, S = JU @ inv, JF @ inv
    A, S = 0.5 * (A + A.mT.contiguous()), 0.5 * (S + S.mT.contiguous())
    L = torch.linalg.cholesky(A)
    Q = torch.linalg.solve_triangular(L, S, upper=False)
    Q = torch.linalg.solve_triangular(L, Q.mT.contiguous(), upper=False)
    lam, E = torch.linalg.eigh((0.5 * (Q + Q.mT.contiguous())).cpu())
    lam, E = lam.to(P.device), E.to(P.device)
    R = L @ E
    dual = torch.linalg.solve_triangular(L.mT.contiguous(), E, upper=True)
    W, v = _thermo(P)[:2]
    near = (lam - v[0][:, None]).abs().argsort(dim=1)[:, :2]
    pick = near[:, None, :].expand(-1, 8, -1)
    two, seed = R.gather(2, pick), dual.gather(2, pick)[:, 0, :]
    w = seed / seed.norm(dim=1, keepdim=True)
    basis = torch.stack([(two * w[:, None, :]).sum(2), two[:, :, 1] * w[:, :1] - two[:, :, 0] * w[:, 1:]], dim=2)
    R = R.scatter(2, pick, basis)
    return lam.T.reshape(8, *shape), R.permute(2, 1, 0).reshape(8, 8, *shape)


def _dissipation(b, P, a):
    """lambda^ T^-1 R Y <<R^T T V>> at faces from the 2p stencil states P and the two metric rows a."""
    p = b.p
    mean = 0.5 * (a[0] + a[1])
    n = torch.cat([mean[1:], torch.zeros_like(mean[:1]).expand(3 - b.dim, *mean.shape[1:])])
    L = torch.sqrt((n * n).sum(0))
    T = _frame(n / L)
    TV = [_turn(T, _entropy(q)) for q in P]
    Vm = 0.5 * (TV[p - 1] + TV[p])
    lam, R = _eigen_rmhd(Vm) if b.rmhd else _eigen_rhd(b, Vm)
    lhat = (mean[0] + L * lam).abs().max(0).values
    scale = TV[p - 1].abs().max(0).values + TV[p].abs().max(0).values
    out = 0.0
    for r in R:
        v = [(r * t).sum(0) for t in TV]
        jump = _weno(v[:0:-1]) - _weno(v[:-1])
        point = v[p] - v[p - 1]
        on = (jump * point > 0) & (point.abs() > 1e-10 * r.abs().sum(0) * scale)
        out = out + torch.where(on, jump, torch.zeros_like(jump)) * r
    return lhat * _turn(T, out, back=True)


def _residual(b, case, P, met):
    """(dU (8 slots), dJ) on the interior from the interior primitive state and the padded metrics."""
    p, ng = b.p, b.ng
    Pp = torch.stack([_extend(b, q, ng, "solution") for q in P])
    dU, dJ = 0.0, 0.0
    for k in range(b.dim):
        Q, a = Pp, met[k]
        for o in range(b.dim):
            if o != k:
                Q, a = _crop(Q, o, ng), _crop(a, o, ng)
        n = b.n[k]
        Ru, Rj, Rs = 0.0, 0.0, 0.0
        for m, al in enumerate(_ALPHA[p], 1):
            # pairs (i, i + m), i = -m .. n - 1
            take = lambda f, lo: _cut(f, k, ng - m + lo, n + m)  # noqa: E731,B023
            F, at, bt = _pair(b, take(Q, 0), take(Q, m), take(a, 0), take(a, m))
            own = lambda f: _cut(f, k, m, n) - _cut(f, k, 0, n)  # noqa: E731,B023
            Ru, Rj = Ru + al * own(F), Rj + al * own(at)
            Rs = Rs + al * own(bt)
        if case["dissipation"]:
            face = lambda f, j: _cut(f, k, ng - 1 + j, n + 1)  # noqa: E731,B023
            d = _dissipation(b, [face(Q, j) for j in range(1 - p, p + 1)], [face(a, 0), face(a, 1)])
            Ru = Ru - 0.5 * (_cut(d, k, 1, n) - _cut(d, k, 0, n))
        if b.rmhd:
            Ru = Ru + _phi_prime(P) * Rs
        dU, dJ = dU - Ru / b.h[k], dJ - Rj / b.h[k]
    return dU[b.slots], dJ


def _fast_speed(b, P):
    """Largest |eigenvalue| of the x flux Jacobian at rotated states."""
    W, v, b0, bv, b2 = _thermo(P)
    rh = P[0] + GAMMA / (GAMMA - 1) * P[4]
    c2 = GAMMA * P[4] / rh
    if not b.rmhd:
        v2, vn = (v * v).sum(0), v[0]
        root = torch.sqrt(c2 * (1 - v2) * (1 - v2 * c2 - vn * vn * (1 - c2)))
        return torch.maximum((vn * (1 - c2) + root).abs(), (vn * (1 - c2) - root).abs()) / (1 - v2 * c2)
    ext = []
    for start in (1.0, -1.0):
        x = torch.full_like(W, start)
        for _ in range(100):
            a, g, e = W * (x - v[0]), 1 - x * x, bv[0] - x * b0
            q = rh * (1 / c2 - 1) * a ** 4 - (rh + b2 / c2) * a * a * g + e * e * g
            dq = (4 * rh * (1 / c2 - 1) * a ** 3 * W - (rh + b2 / c2) * (2 * a * W * g - 2 * a * a * x)
                  - 2 * e * b0 * g - 2 * e * e * x)
            s = q / dq
            x = torch.where(s * start > 0, x - s, x)
        ext.append(x.abs())
    return torch.maximum(*ext)


def _time_step(b, case, P, met, J):
    total = 0.0
    for k in range(b.dim):
        a = _inner(b, met[k])[1:]
        n = torch.cat([a, torch.zeros_like(a[:1]).expand(3 - b.dim, *a.shape[1:])])
        L = torch.sqrt((n * n).sum(0))
        total = total + float((L * _fast_speed(b, _turn(_frame(n / L), P)) / J).max()) / b.h[k]
    return case["cfl"] / total


def _redistribute(b, case, P, x, dt):
    """(x_new, xdot): monitor, three filter passes, Jacobi sweeps and the move limiter."""
    d, one = b.dim, lambda f, rule, c=-1: _extend(b, f, 1, rule, c)  # noqa: E731

    def nb(fe, k, s):
        for o in range(d):
            fe = _cut(fe, o, 1 + (s if o == k else 0), b.n[o])
        return fe

    free = []
    for k in range(d):
        i = torch.arange(b.n[k], device=x.device)
        f = torch.ones_like(i, dtype=torch.bool) if b.periodic[k] else (i > 0) & (i < b.n[k] - 1)
        free.append(f.reshape([-1 if a == d - 1 - k else 1 for a in range(d)]))
    s = torch.log(P[0]) if case["sigma"] else P[0]
    se = one(s, "solution")
    g2, lap = 0.0, 0.0
    for k in range(d):
        up, dn = nb(se, k, 1), nb(se, k, -1)
        # the edge copy makes the difference one-sided on bounded edges, over one spacing instead of two
        g2 = g2 + ((up - dn) / (b.h[k] * (1.0 + free[k].to(up.dtype)))) ** 2
        second = up - 2 * s + dn
        if not b.periodic[k]:
            ax = _axis(second, k)
            i = torch.arange(b.n[k], device=x.device).clamp(1, b.n[k] - 2)
            second = second.index_select(ax, i)
        lap = lap + second / b.h[k] ** 2
    if case["form"] == 1:
        w = torch.sqrt(1 + case["alpha"] * g2)
    else:
        g = torch.sqrt(g2)
        w = 1 + case["alpha"] * g / g.max() if g.max() > 0 else torch.ones_like(g)
        if case["form"] == 2 and lap.abs().max() > 0:
            w = w + 0.5 * case["alpha"] * lap.abs() / lap.abs().max()
        w = torch.sqrt(w)
    for _ in range(3):
        for k in range(d):
            we = one(w, "solution")
            w = 0.25 * (nb(we, k, 1) + nb(we, k, -1)) + 0.5 * w
    we = one(w, "solution")
    y = x.clone()
    for _ in range(case["sweeps"]):
        den, num = 0.0, [0.0] * d
        for k in range(d):
            cp, cm = (torch.where(free[k], w + nb(we, k, q), torch.zeros_like(w)) for q in (1, -1))
            den = den + cp + cm
            for c in range(d):
                ye = one(y[c], "mesh", c)
                num[c] = num[c] + cp * nb(ye, k, 1) + cm * nb(ye, k, -1)
        y = torch.stack([torch.where(free[c] & (den > 0), num[c] / torch.where(den > 0, den, 1.0), y[c])
                         for c in range(d)])
    dx = y - x
    tau = torch.ones((), dtype=x.dtype, device=x.device)
    for k in range(d):
        xe = one(x[k], "mesh", k)
        gap = torch.where(dx[k] < 0, nb(xe, k, -1) - x[k], nb(xe, k, 1) - x[k])
        tau = torch.minimum(tau, torch.where(dx[k] != 0, gap / (2 * dx[k]), torch.ones_like(gap)).min())
    return x + tau * dx, tau * dx / dt


def _step(b, case, U, J, x, xdot, dt):
    """One step; xdot given, or None for the case's own mesh rule.  The mesh and dt carry no gradient."""
    P = _recover(b, U, J)
    with torch.no_grad():
        if dt is None:
            dt = _time_step(b, case, P, _metrics(b, x), J)
        if xdot is not None:
            x1 = x + dt * xdot
        elif case["form"] >= 0:
            x1, xdot = _redistribute(b, case, P.detach(), x, dt)
        else:
            x1, xdot = x, torch.zeros_like(x)
    Us, Js = U, J
    for s, c in enumerate((0.0, 1.0, 0.5)):
        if s:
            P = _recover(b, Us, Js)
        L, LJ = _residual(b, case, P, _metrics(b, x + c * dt * xdot, xdot))
        w = (0.0, 0.75, 1.0 / 3.0)[s]
        Us, Js = w * U + (1 - w) * (Us + dt * L), w * J + (1 - w) * (Js + dt * LJ)
    return Us, Js, x1, xdot, torch.full((1,), dt, dtype=torch.float64, device=x.device)


def _has_exact(case):
    if case["mixed"] and case["do"] != "residual":
        return False
    if case["phys"] == "rmhd" and case["dissipation"] and case["do"] in ("residual", "step", "adjoint"):
        # one small eigenproblem per face and stage
        return case["flow"] == "smooth" and math.prod(_Box(case).n) * case["dim"] <= 140_000
    return True


def exact(case, seed):
    if not _has_exact(case):
        return None
    b, P, x, xdot = _inputs(case, seed)
    do = case["do"]
    J = _jacobian(b, x)
    U = (J * _conserved(P))[b.slots]
    if do == "setup":
        return torch.cat(_metrics(b, x)), J, U
    if do == "recover":
        met = _metrics(b, x)
        P = _recover(b, U, J)
        rows = [P[c] for c in b.slots] + [torch.log(P[0]), torch.log(P[0] / P[4])]
        dt = _time_step(b, case, P, met, J)
        return (torch.stack([_extend(b, r, b.ng, "solution") for r in rows]),
                torch.full((1,), dt, dtype=torch.float64, device="cuda"))
    if do == "residual":
        return _residual(b, case, _recover(b, U, J), _metrics(b, x, xdot))
    if do == "step":
        return _step(b, case, U, J, x, None, None)
    if do == "moving":
        return _step(b, case, U, J, x, xdot, _vortex_dt(b))[:3]
    U, J = U.requires_grad_(), J.requires_grad_()
    out = _step(b, case, U, J, x, None, None if case["form"] >= 0 else _adjoint_dt(b))
    gU, gJ = torch.autograd.grad(out[:2], (U, J), _cotangents(b, seed))
    return out[0].detach(), out[1].detach(), out[2], out[4], gU, gJ
