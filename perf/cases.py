"""Performance cases of the solver: what a program has it do, through the public entry points.

A program advances a state by Strang steps (dt from the positivity CFL rule before each), or one of
the two subflows alone, or an ensemble of runs together, or differentiates the two right-hand sides
through torch.autograd.  Every array is float64, the only type the library has.

``exact`` is the scheme in plain torch: tensor-product tables from numpy's Legendre routines, loops
over node pairs, and torch.autograd for the gradients."""
import math
import random

import numpy as np
import torch
from numpy.polynomial import legendre as npleg

import paper_2609_10849_amd as pk
from paper_2609_10849_amd import autograd as ag

GAMMA = 5.0 / 3.0
CFL = 0.3
DEV = "cuda" if torch.cuda.is_available() else "cpu"

# ---------------------------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------------------------


def _case(kind, flow, nx, ny, p, m, stab="full", walls=0, reduced=0, order=0):
    return dict(kind=kind, flow=flow, nx=nx, ny=ny, p=p, m=m, stab=stab, walls=walls, reduced=reduced, order=order)


def listed():
    return [
        # a small convergence-study run: a few kernels of one wave each, so latency and launches
        dict(_case("step", "vortex", 16, 16, 3, 2, "none"), name="step_vortex_16x16_p3"),
        # a row of the stabilised-vortex study
        dict(_case("step", "vortex", 64, 64, 2, 2), name="step_vortex_64x64_p2"),
        # the nonsmooth experiments' mesh and degree (Orszag-Tang, blast), every stabiliser on
        dict(_case("step", "orszag", 256, 256, 2, 2), name="step_orszag_256x256_p2"),
        # the rotor between mirror walls: the mirror-doubled mesh, amplitudes over the box
        dict(_case("step", "rotor", 512, 512, 2, 2, walls=3), name="step_rotor_512x512_p2_walls"),
        # a high degree on an odd, not square mesh, all eight variables nonzero
        dict(_case("step", "mixed", 241, 137, 5, 4), name="step_mixed_241x137_p5"),
        # a 2D2V state through the reduced system
        dict(_case("step", "orszag", 512, 512, 4, 3, reduced=1), name="step_orszag_512x512_p4_2d2v"),
        # the benchmark's state: a large production step
        dict(_case("step", "blast", 1024, 1024, 4, 3), name="step_blast_1024x1024_p4"),
        # the hydro subflow alone (Euler runs), oscillation elimination and positivity scaling
        dict(_case("hydro", "mixed", 512, 512, 3, 2, "oe"), name="hydro_mixed_512x512_p3"),
        # the magnetic subflow alone: the largest run of the reduced Alfven-wave study
        dict(_case("magnetic", "alfven", 128, 128, 4, 4, "none"), name="magnetic_alfven_128x128_p4"),
        # sensitivities: forward and backward of both right-hand sides, ordinary and large
        dict(_case("adjoint", "noisy", 128, 128, 3, 2, "none"), name="adjoint_noisy_128x128_p3"),
        dict(_case("adjoint", "mixed", 1024, 1024, 4, 3, "none"), name="adjoint_mixed_1024x1024_p4"),
        # an ensemble of 64 uneven runs advanced together, its step replayed from a graph
        dict(kind="ensemble", runs=64, table=0, largest=192, name="ensemble_64_runs"),
    ]


def draw(rng):
    kind = rng.choices(["step", "hydro", "magnetic", "adjoint", "ensemble"], [50, 12, 12, 14, 12])[0]
    if kind == "ensemble":
        return dict(kind=kind, runs=rng.randint(4, 48), table=rng.randint(1, 10 ** 6), largest=rng.choice([64, 96, 128, 192]))
    p = rng.choices([1, 2, 3, 4, 5, 6], [8, 25, 25, 25, 10, 7])[0]
    m = p - rng.randint(0, 1)
    n = math.exp(rng.uniform(math.log(12.0), math.log(1024.0)))
    # the table of the velocity projection grows as (p+1)^4 per element: no larger than the largest listed one's
    n = min(n, math.sqrt(0.55 * 1024 ** 2 * (25.0 / (p + 1) ** 2) ** 2))
    a = 2.0 ** rng.uniform(-0.75, 0.75)
    nx, ny = max(8, int(n * a)), max(8, int(n / a))
    stab, walls, reduced, order = "full", 0, 0, 0
    if kind == "adjoint":
        flow, stab = rng.choice(["noisy", "mixed"]), "none"
    elif kind == "magnetic":
        flow, stab = rng.choice([("alfven", "none"), ("mixed", "full")])
    elif kind == "hydro":
        flow, stab = rng.choice([("vortex", "none"), ("mixed", "oe")])
    else:
        flow, stab = rng.choice([("vortex", "none"), ("vortex", "full"), ("orszag", "full"), ("orszag", "oe"), ("blast", "full"), ("mixed", "full"), ("rotor", "full")])
        reduced = rng.randint(0, 1) if flow == "orszag" else 0
        order = rng.choice([0, 0, 0, 1])
    if flow == "rotor":
        walls, nx, ny = 3, 2 * ((nx + 1) // 2), 2 * ((ny + 1) // 2)
    return _case(kind, flow, nx, ny, p, m, stab, walls, reduced, order)


def _members(case):
    """The runs of an ensemble as cases of their own: uneven meshes and degrees from its table number."""
    r = random.Random(case["table"])
    sizes = [n for n in (32, 64, 96, 128, 192) if n <= case["largest"]]
    out = []
    for _ in range(case["runs"]):
        n, p = r.choice(sizes), r.choice([2, 3, 4])
        out.append(_case("step", "vortex", n, n, p, p - 1))
    return out


# ---------------------------------------------------------------------------------------------
# Initial states
# ---------------------------------------------------------------------------------------------


def _gll(r):
    if r == 0:
        return np.array([0.0]), np.array([2.0])
    x = np.concatenate([[-1.0], np.sort(npleg.Legendre.basis(r).deriv().roots().real), [1.0]])
    return x, 2.0 / (r * (r + 1) * npleg.legval(x, [0.0] * r + [1.0]) ** 2)


def _basis(src, dst, deriv=0):
    """[dst][src]: the deriv-th derivatives at dst of the Lagrange basis of the nodes src."""
    c = np.linalg.solve(npleg.legvander(src, len(src) - 1), np.eye(len(src)))
    return npleg.legval(dst, npleg.legder(c, deriv) if deriv else c).T if deriv < len(src) else np.zeros((len(dst), len(src)))


DOMAIN = {"vortex": (0.0, 10.0), "noisy": (0.0, 10.0), "alfven": (0.0, 2 * math.pi), "orszag": (0.0, 2 * math.pi),
          "mixed": (0.0, 1.0), "blast": (-0.5, 0.5), "rotor": (0.0, 2.0)}


class _Mesh:
    def __init__(self, case):
        self.nx, self.ny, self.p, self.m = (int(case[k]) for k in ("nx", "ny", "p", "m"))
        self.lo, self.hi = DOMAIN[case["flow"]]
        self.walls = int(case["walls"])
        self.hx, self.hy = (self.hi - self.lo) / self.nx, (self.hi - self.lo) / self.ny
        self.bx = self.nx // 2 if self.walls & 1 else self.nx
        self.by = self.ny // 2 if self.walls & 2 else self.ny
        self.np, self.K = self.p + 1, self.nx * self.ny
        self.xp, self.wp = _gll(self.p)
        self.xw, self.ww = _gll(self.m + 1)
        self.xv, _ = _gll(self.m)
        self.xg, self.wg = npleg.leggauss(self.m + 1)
        self.xq, self.wq = npleg.leggauss(self.m + 2)

    def tab(self, a):
        return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)

    def _axis(self, n, h, s):
        return self.tab(self.lo + (np.arange(n)[:, None] + 0.5 * (s[None, :] + 1.0)) * h)

    def u_nodes(self):  # [ny, nx, j, i]
        X, Y = self._axis(self.nx, self.hx, self.xp), self._axis(self.ny, self.hy, self.xp)
        shape = (self.ny, self.nx, self.np, self.np)
        return X[None, :, None, :].expand(shape), Y[:, None, :, None].expand(shape)

    def grid(self, sx, sy):  # [ny (m+1), nx (m+1)]
        X, Y = self._axis(self.nx, self.hx, sx).reshape(-1), self._axis(self.ny, self.hy, sy).reshape(-1)
        return X[None, :].expand(len(Y), -1), Y[:, None].expand(-1, len(X))

    def w_grid(self):
        return self.grid(self.xw[:-1], self.xw[:-1])

    def local(self, g, wide_x, wide_y):
        """[ny, nx, j, i] values of a grid; a wide direction has the next element's first node too."""
        M1 = self.m + 1
        g = g.reshape(self.ny, M1, self.nx, M1).permute(0, 2, 1, 3)
        if wide_x:
            g = torch.cat([g, torch.roll(g, -1, 1)[..., :1]], -1)
        if wide_y:
            g = torch.cat([g, torch.roll(g, -1, 0)[..., :1, :]], -2)
        return g

    def to_grid(self, loc):
        M1 = self.m + 1
        return loc[..., :M1, :M1].permute(0, 2, 1, 3).reshape(self.ny * M1, self.nx * M1).contiguous()

    def curl(self, A):
        """The in-plane field (-d_y A, d_x A) of a potential on the shared GLL_{m+1} nodes."""
        L = self.local(A, True, True)
        D = self.tab(_basis(self.xw, self.xg, 1))
        return self.to_grid(-_ay(L, D) * (2.0 / self.hy)), self.to_grid(_ax(L, D) * (2.0 / self.hx))


def _ax(x, T):
    """T applied along the last index."""
    return (x.reshape(-1, x.shape[-1]) @ T.t().contiguous()).reshape(*x.shape[:-1], T.shape[0])


def _ay(x, T):
    """T applied along the last index but one."""
    return _ax(x.transpose(-1, -2).contiguous(), T).transpose(-1, -2)


def _axy(x, Tx, Ty):
    return _ay(_ax(x, Tx), Ty)


def _pack(rho, u, p):
    E = p / (GAMMA - 1.0) + 0.5 * rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])
    return torch.stack([rho, rho * u[0], rho * u[1], rho * u[2], E])


def _initial(case, seed):
    """(mesh, U [5, K, p+1, p+1], Bx, By, Bz) of a flow; the seed moves and scales it."""
    M, r = _Mesh(case), random.Random(seed)
    X, Y = M.u_nodes()
    WX, WY = M.w_grid()
    zero, size = torch.zeros_like(X), M.hi - M.lo
    gshape = (M.ny * (M.m + 1), M.nx * (M.m + 1))
    full = lambda v: torch.full(gshape, float(v), dtype=torch.float64, device=DEV)  # noqa: E731
    flow = case["flow"]
    if flow in ("vortex", "noisy"):  # an isentropic vortex, the peak swirl and the field as the ensemble draws them
        kappa, cx, cy = r.uniform(0.1, 0.8), M.lo + size * r.uniform(0.3, 0.7), M.lo + size * r.uniform(0.3, 0.7)
        b, ang = r.uniform(0.05, 0.3), r.uniform(0.0, 2 * math.pi)
        wrap = lambda d: d - size * torch.round(d / size)  # noqa: E731
        dx, dy = wrap(X - cx), wrap(Y - cy)
        r2 = dx * dx + dy * dy
        s = kappa * torch.exp(0.5 * (1.0 - r2))
        T = 1.0 - (GAMMA - 1.0) / GAMMA * 0.5 * kappa ** 2 * torch.exp(1.0 - r2)
        rho = T ** (1.0 / (GAMMA - 1.0))
        U = _pack(rho, (-s * dy, s * dx, zero), rho * T)
        Bx, By, Bz = full(b * math.cos(ang)), full(b * math.sin(ang)), full(0.0)
        if flow == "noisy":  # noise of 1e-3 on every value, the in-plane field's through a potential
            g = torch.Generator(DEV).manual_seed(seed)
            noise = lambda t: 1e-3 * torch.randn(t.shape, dtype=torch.float64, device=DEV, generator=g)  # noqa: E731
            U = U + noise(U)
            dBx, dBy = M.curl(noise(Bx))
            Bx, By, Bz = Bx + M.hx * dBx, By + M.hx * dBy, Bz + noise(Bz)
    elif flow == "alfven":  # a circularly polarised Alfven wave along (1, 1)
        eps, ph, q = r.uniform(0.05, 0.2), r.uniform(0.0, 2 * math.pi), math.sqrt(0.5)
        wave = lambda x, y: torch.cos(x + y + ph)  # noqa: E731
        c, s = eps * wave(X, Y), eps * torch.sin(X + Y + ph)
        U = _pack(torch.ones_like(X), (q * c, -q * c, -s), torch.ones_like(X))
        Bx = q - q * eps * wave(*M.grid(M.xw[:-1], M.xg))
        By = q + q * eps * wave(*M.grid(M.xg, M.xw[:-1]))
        vx, vy = M.grid(M.xv, M.xv)
        Bz = eps * torch.sin(vx + vy + ph)
    elif flow == "orszag":  # the Orszag-Tang vortex, its origin moved
        a, b = r.uniform(0.0, 2 * math.pi), r.uniform(0.0, 2 * math.pi)
        U = _pack(torch.full_like(X, GAMMA * GAMMA), (-torch.sin(Y + b), torch.sin(X + a), zero), torch.full_like(X, GAMMA))
        Bx, By = M.curl(-torch.cos(WY + b) - 0.5 * torch.cos(2.0 * (WX + a)))
        Bz = full(0.0)
    elif flow == "blast":  # an over-pressured disc in a uniform oblique field
        cx, cy, ang = r.uniform(-0.1, 0.1), r.uniform(-0.1, 0.1), r.uniform(0.2, 1.3)
        inside = (X - cx) ** 2 + (Y - cy) ** 2 < 0.01
        U = _pack(torch.ones_like(X), (zero, zero, zero), torch.where(inside, torch.full_like(X, 1000.0), torch.full_like(X, 0.1)))
        Bx, By, Bz = full(math.cos(ang)), full(math.sin(ang)), full(0.0)
    elif flow == "rotor":  # a spinning dense disc in the box [0, 1]^2 and its mirror images
        spin, field = r.uniform(0.6, 1.0), r.uniform(0.5, 0.75)
        fold = lambda v: (torch.where(v <= 1.0, v, 2.0 - v) - 0.5, torch.where(v <= 1.0, 1.0, -1.0))  # noqa: E731
        (dx, sx), (dy, sy) = fold(X), fold(Y)
        rr = torch.sqrt(dx * dx + dy * dy)
        f = torch.clamp((0.115 - rr) / 0.015, 0.0, 1.0)
        rho = torch.where(rr < 0.1, torch.full_like(rr, 10.0), 1.0 + 9.0 * f)
        w = spin * torch.where(rr < 0.1, rr / 0.1, f) / torch.clamp(rr, min=1e-30)
        U = _pack(rho, (-sx * w * dy, sy * w * dx, zero), torch.full_like(X, 0.5))
        Bx, By, Bz = full(field), full(0.0), full(0.0)
    else:  # "mixed": subsonic turbulence, a few random waves in every variable
        two_pi = 2 * math.pi / size

        def waves(x, y, amp):
            v = torch.zeros_like(x)
            for _ in range(4):
                v = v + amp * r.uniform(0.2, 0.5) * torch.sin(two_pi * (r.randint(-3, 3) * x + r.randint(1, 3) * y) + r.uniform(0.0, 6.28))
            return v

        rho, pr = 1.0 + waves(X, Y, 0.15), 1.0 + waves(X, Y, 0.15)
        U = _pack(rho, (waves(X, Y, 0.3), waves(X, Y, 0.3), waves(X, Y, 0.2)), pr)
        Bx, By = M.curl(waves(WX, WY, 0.05 * size))
        Bx, By, Bz = Bx + 0.3, By + 0.2, waves(*M.grid(M.xv, M.xv), 0.2)
    return (M, U.reshape(5, M.K, M.np, M.np).contiguous()) + tuple(t.contiguous() for t in (Bx, By, Bz))


def _cotangents(case, seed, M, U, Bx):
    """Cotangents of L_E and L_M and a resistivity, as a gradient step brings them in."""
    g = torch.Generator(DEV).manual_seed(seed + 7)
    normal = lambda *s: torch.randn(s, dtype=torch.float64, device=DEV, generator=g)  # noqa: E731
    sh = tuple(U.shape[1:])
    eta = 1e-3 * torch.rand(M.K, dtype=torch.float64, device=DEV, generator=g)
    return eta, normal(*U.shape), [normal(*sh), normal(3, *sh)] + [normal(*Bx.shape) for _ in range(3)]


# ---------------------------------------------------------------------------------------------
# What a program has in hand, and one pass
# ---------------------------------------------------------------------------------------------


def _options(case):
    on = {"none": (0, 0, 0, 0), "oe": (1, 1, 1, 0), "full": (1, 1, 1, 1)}[case["stab"]]
    return pk.Options.make(*on, reduced_2d2v=case["reduced"], strang_order=case["order"])


class _Run:
    """One run's layout, as pk.Batch takes it."""

    def __init__(self, case):
        M = _Mesh(case)
        self.nx, self.ny, self.p, self.m, self.walls, self.gamma = M.nx, M.ny, M.p, M.m, M.walls, GAMMA
        self.x0 = self.y0 = M.lo
        self.x1 = self.y1 = M.hi


def _flat(states, k):
    """One buffer holding the k-th array of every state, and its views."""
    flat = torch.cat([s[k].reshape(-1) for s in states])
    views, at = [], 0
    for s in states:
        views.append(flat[at:at + s[k].numel()].view(s[k].shape))
        at += s[k].numel()
    return flat, views


def prepare(case, seed):
    if case["kind"] == "ensemble":
        members = _members(case)
        states = [_initial(c, seed + 1000 * i)[1:] for i, c in enumerate(members)]
        dts = []
        for c, s in zip(members, states):
            S = pk.Solver.from_layout(_Run(c), _options(c))
            dts.append(S.cfl_dt(*s, CFL))
            S.close()
        arrays = [_flat(states, k) for k in range(4)]
        B = pk.Batch([_Run(c) for c in members], _options(members[0]))
        B.graph(True)
        return dict(kind="ensemble", B=B, flat=[a[0] for a in arrays], views=[a[1] for a in arrays], dts=dts)
    M, U, Bx, By, Bz = _initial(case, seed)
    S = pk.Solver.from_layout(_Run(case), _options(case))
    st = dict(kind=case["kind"], S=S, g=[U, Bx, By, Bz])
    if case["kind"] == "hydro":
        st["tau"] = 0.5 * S.cfl_dt(U, Bx, By, Bz, CFL)
    elif case["kind"] == "magnetic":
        st["tau"] = S.cfl_dt(U, Bx, By, Bz, CFL)
        st["prim"] = S.to_primitive(U)
    elif case["kind"] == "adjoint":
        eta, cot, cots = _cotangents(case, seed, M, U, Bx)
        rho, _, u = S.to_primitive(U)
        st.update(eta=eta, cot=cot, cots=cots, rho=rho, leaf=[t.requires_grad_() for t in (u, Bx, By, Bz)])
        st["g"][0] = U.requires_grad_()
    return st


def _ok(status):
    if status:
        raise RuntimeError("step refused: %d" % status)


def run(state):
    kind = state["kind"]
    if kind == "ensemble":  # as a program that steps its runs at fixed steps does
        r, _ = state["B"].strang_step(*state["views"], state["dts"])
        _ok(r)
        return state["flat"]
    S, g = state["S"], state["g"]
    if kind == "step":
        dt = S.cfl_dt(*g, CFL)
        r, _ = S.strang_step(*g, dt)
        _ok(r)
        return [*g, dt]
    if kind == "hydro":
        r, _ = S.hydro_substep(g[0], state["tau"])
        _ok(r)
        return [g[0]]
    if kind == "magnetic":
        rho, e, u = state["prim"]
        rep = S.step_magnetic(rho, e, u, g[1], g[2], g[3], state["tau"])
        _ok(rep["status"])
        return [e, u, g[1], g[2], g[3]]
    dU = ag.rhs_hydro(S, g[0])
    grad, = torch.autograd.grad(dU, g[0], state["cot"])
    out = ag.rhs_magnetic(S, state["rho"], *state["leaf"], eta=state["eta"])
    grads = torch.autograd.grad(out, state["leaf"], state["cots"])
    return [dU.detach(), grad, *(t.detach() for t in out), *grads]


def work(case):
    """Bytes: the state in and out once (the adjoint: inputs, cotangents, outputs and gradients).
    Flops: what the stages' formulas take (an EC flux 74 per node pair, a face flux 50, the transforms
    and interpolations as sums over one index at a time)."""
    if case["kind"] == "ensemble":
        each = [work(c) for c in _members(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    K, n, B, A = case["nx"] * case["ny"], case["p"] + 1, case["m"] + 1, case["m"] + 2
    nn, oe = n * n, case["stab"] != "none"
    hydro = nn * (65 + 74 * (n - 1)) + 160 * n + (oe and 10 * n * (4 * nn + 3 * n) + 40 * n ** 3 + 40 * nn)
    mag = 8 * A * A * (A + B) + 6 * nn * (A + B) + 8 * n * A * (n + A) * 3 + 60 * nn
    vel = oe and 6 * n * (4 * nn + 3 * n) + 12 * nn * nn + 30 * nn
    prep = oe and nn ** 3
    U, G = 5 * nn * 8, 3 * B * B * 8
    if case["kind"] == "step":
        return {"bytes": K * 2.0 * (U + G), "flops": K * (6.0 * hydro + 3 * (mag + vel) + prep)}
    if case["kind"] == "hydro":
        return {"bytes": K * 2.0 * U, "flops": K * 3.0 * hydro}
    if case["kind"] == "magnetic":
        return {"bytes": K * (nn * 8.0 + 2 * (4 * nn * 8 + G)), "flops": K * (3.0 * (mag + vel) + prep)}
    return {"bytes": K * (4.0 * U + 5 * G + 15 * nn * 8), "flops": K * 3.0 * (hydro + mag)}


# ---------------------------------------------------------------------------------------------
# The scheme in plain torch.  Arrays: U [5, ny, nx, j, i]; magnetic fields as grids.
# ---------------------------------------------------------------------------------------------
EPS = 2.0 ** -52


def _pressure(s):
    return (GAMMA - 1.0) * (s[4] - 0.5 * (s[1] * s[1] + s[2] * s[2] + s[3] * s[3]) / s[0])


def _logmean(a, b):
    f = (b - a) / (a + b)
    near = f.abs() < 0.05
    u = f * f
    s = torch.full_like(f, 1.0 / 21.0)
    for k in range(9, -1, -1):
        s = s * u + 1.0 / (2 * k + 1)
    q = torch.where(near, torch.full_like(f, 2.0), b / a)
    return torch.where(near, 0.5 * (a + b) / s, (b - a) / torch.log(q))


def _phys(s, d):
    ud, p = s[1 + d] / s[0], _pressure(s)
    f = [s[1 + d], s[1] * ud, s[2] * ud, s[3] * ud, (s[4] + p) * ud]
    f[1 + d] = f[1 + d] + p
    return torch.stack(f)


def _ec(a, b, d):
    ua, ub = a[1:4] / a[0], b[1:4] / b[0]
    ba, bb = a[0] / (2.0 * _pressure(a)), b[0] / (2.0 * _pressure(b))
    rlog, blog, um = _logmean(a[0], b[0]), _logmean(ba, bb), 0.5 * (ua + ub)
    phat = 0.5 * (a[0] + b[0]) / (ba + bb)
    h = 1.0 / (2.0 * (GAMMA - 1.0) * blog) - 0.25 * ((ua * ua).sum(0) + (ub * ub).sum(0)) + (um * um).sum(0) + phat / rlog
    f = [rlog * um[d]] + [rlog * um[k] * um[d] for k in range(3)] + [rlog * um[d] * h]
    f[1 + d] = f[1 + d] + phat
    return torch.stack(f)


def _llf(a, b, d):
    speed = lambda s: (s[1 + d] / s[0]).abs() + torch.sqrt(GAMMA * _pressure(s) / s[0])  # noqa: E731
    return 0.5 * (_phys(a, d) + _phys(b, d)) - 0.5 * torch.maximum(speed(a), speed(b)) * (b - a)


def _hydro_terms(M, U):
    """The terms of L_E one after another: (nodes along the line, coefficients, flux, direction)."""
    D, p = _basis(M.xp, M.xp, 1), M.p
    for d, h in ((0, M.hx), (1, M.hy)):
        at = lambda i: (U if d == 0 else U.transpose(-1, -2))[..., i]  # noqa: E731
        face = lambda: _llf(torch.roll(at(p), 1, 2 - d), at(0), d)  # noqa: E731
        for i in range(M.np):
            yield d, [(i, -4.0 / h * D[i, i])], _phys(at(i), d)
            for r in range(i):
                yield d, [(i, -4.0 / h * D[i, r]), (r, -4.0 / h * D[r, i])], _ec(at(i), at(r), d)
        yield d, [(0, 2.0 / (h * M.wp[0]))], face() - _phys(at(0), d)
        yield d, [(p, 2.0 / (h * M.wp[p]))], _phys(at(p), d) - torch.roll(face(), -1, 2 - d)


def _rhs_hydro(M, U):
    out = torch.zeros_like(U)
    for d, at, f in _hydro_terms(M, U):
        V = out if d == 0 else out.transpose(-1, -2)
        for i, c in at:
            V[..., i] += c * f
    return out


def _rhs_hydro_vjp(M, U, cot):
    grad = torch.zeros_like(U)
    U = U.detach().requires_grad_()
    for d, at, f in _hydro_terms(M, U):
        C = cot if d == 0 else cot.transpose(-1, -2)
        g, = torch.autograd.grad(f, U, sum(c * C[..., i] for i, c in at))
        grad += g
    return grad


def _amplitudes(M, w, average):
    """Global and line amplitudes of one field over the box: (row [ny, 1], column [1, nx], constant)."""
    hi, lo = w.amax((-1, -2)), w.amin((-1, -2))
    box = (slice(0, M.by), slice(0, M.bx))
    dev = lambda mean, dims, sl: torch.maximum((hi[sl].amax(dims) - mean).abs(), (lo[sl].amin(dims) - mean).abs())  # noqa: E731
    dom = dev(average[box].mean(), (0, 1), box)
    row = dev(average[:, :M.bx].mean(1), (1,), (slice(None), slice(0, M.bx)))
    col = dev(average[:M.by].mean(0), (0,), (slice(0, M.by),))
    top, bot = hi[box].max(), lo[box].min()
    const = bool(top - bot <= 1024.0 * EPS * torch.maximum(top.abs(), bot.abs()))
    return torch.maximum(row, 1e-6 * dom)[:, None], torch.maximum(col, 1e-6 * dom)[None, :], const


def _average(M, w):
    W = M.tab(np.outer(M.wp, M.wp) / 4.0)
    return (w * W).sum((-1, -2))


def _sensor(M, fields):
    """sigma[direction][order], each [ny, nx], of fields that share their amplitude."""
    amp = [_amplitudes(M, w, _average(M, w)) for w in fields]
    out = []
    for d, h in ((0, M.hx), (1, M.hy)):
        shared = torch.stack([a[d] for a in amp]).amax(0)
        sig = [torch.zeros(M.ny, M.nx, dtype=torch.float64, device=DEV) for _ in range(M.np)]
        for w, a in zip(fields, amp):
            if a[2]:
                continue
            V = w if d == 0 else w.transpose(-1, -2)
            for r in range(M.np):
                ends = _ax(V.contiguous(), M.tab(_basis(M.xp, np.array([-1.0, 1.0]), r)))
                jump = ends[..., 0] - torch.roll(ends[..., 1], 1, 1 - d)
                s = torch.sqrt((jump * jump * M.tab(0.5 * M.wp)).sum(-1)) * (2.0 / h) ** r
                J = s + torch.roll(s, -1, 1 - d)
                v = (2 * r + 1) * h ** r / (2.0 * math.factorial(r)) * J / shared
                sig[r] = torch.maximum(sig[r], torch.where(shared > 0, v, torch.zeros_like(v)))
        out.append(sig)
    return out


def _damping(M, sig, lam, s_tau):
    D, total = [torch.ones_like(lam[0])], lam[0] * sig[0][0] + lam[1] * sig[1][0]
    for r in range(1, M.np):
        total = total + lam[0] * sig[0][r] + lam[1] * sig[1][r]
        D.append(torch.exp(-s_tau * total))
    return D


def _hydro_map(M, U, tau):
    avg = _average(M, U)
    # oscillation elimination: the discrete Legendre modes damped by shells
    c = torch.sqrt(GAMMA * _pressure(avg) / avg[0])
    lam = [(2 * M.p + 1) * ((avg[1 + d] / avg[0]).abs() + c) / h for d, h in ((0, M.hx), (1, M.hy))]
    D = _damping(M, _sensor(M, list(U)), lam, 0.02 * tau)
    V = npleg.legvander(M.xp, M.p)
    T = M.tab(np.linalg.inv(V))
    shell = [[max(a, b) for a in range(M.np)] for b in range(M.np)]
    F = torch.stack([torch.stack([D[l] for l in row], -1) for row in shell], -2)
    U = _axy(_axy(U, T, T) * F, M.tab(V), M.tab(V))
    # positivity scaling
    a, e_r = avg[..., None, None], 64.0 * EPS
    low = U[0].amin((-1, -2))
    th = torch.where(low < e_r, ((avg[0] - e_r) / (avg[0] - low)).clamp(0.0, 1.0), torch.ones_like(low))[..., None, None]
    U = torch.cat([torch.where(th < 1.0, a[0] + th * (U[0] - a[0]), U[0])[None], U[1:]])
    size = lambda s: s[4].abs() + 0.5 * (s[1] * s[1] + s[2] * s[2] + s[3] * s[3]) / s[0].clamp(min=e_r)  # noqa: E731
    e_p = (8192.0 * EPS * torch.maximum(size(U).amax((-1, -2)), size(avg))).clamp(min=64.0 * EPS)
    pbar, low = _pressure(avg), _pressure(U).amin((-1, -2))
    th = torch.where(low < e_p, ((pbar - e_p) / (pbar - low)).clamp(0.0, 1.0), torch.ones_like(low))
    th = torch.where((pbar <= e_p) | (avg[0] <= e_r), torch.zeros_like(th), th)[..., None, None]
    return torch.where(th < 1.0, a + th * (U - a), U)


def _hydro(M, case, U, tau):
    def stage(a, b, S):
        Y = a * U + b * (S + tau * _rhs_hydro(M, S))
        return _hydro_map(M, Y, tau) if case["stab"] != "none" else Y

    S = stage(0.0, 1.0, U)
    S = stage(0.75, 0.25, S)
    return stage(1.0 / 3.0, 2.0 / 3.0, S)


def _fields(M, B):
    """The local nodal values of (Bx, By, Bz) with their node sets."""
    return [(M.local(B[0], True, False), M.xw, M.xg), (M.local(B[1], False, True), M.xg, M.xw), (M.local(B[2], False, False), M.xv, M.xv)]


def _at(M, field, X, Y, dx=0, dy=0):
    v, xs, ys = field
    v = _axy(v, M.tab(_basis(xs, X, dx)), M.tab(_basis(ys, Y, dy)))
    return v * (2.0 / M.hx if dx else 1.0) * (2.0 / M.hy if dy else 1.0)


def _assemble(M, loc, wx, wy, J):
    """Sum the local loads of shared nodes and divide by their lumped weights; also the local values."""
    w = M.tab(np.outer(wy, wx) * J).expand(loc.shape)
    for wide, dim, cut in ((len(wx) == M.m + 2, 1, -1), (len(wy) == M.m + 2, 0, -2)):
        if wide:
            n = loc.shape[cut]
            out = []
            for t in (loc, w):
                first = t.narrow(cut, 0, 1) + torch.roll(t.narrow(cut, n - 1, 1), 1, dim)
                out.append(torch.cat([first, t.narrow(cut, 1, n - 2)], cut))
            loc, w = out
    return M.to_grid(loc / w)


def _rhs_magnetic(M, rho, u, B, eta):
    J0 = M.hx * M.hy / 4.0
    F = _fields(M, B)
    W, Gs, Q, P = M.xw, M.xg, M.xq, M.xp
    wq, wg = M.tab(np.outer(M.wq, M.wq) * J0), M.tab(np.outer(M.wg, M.wg) * J0)
    T = lambda src, dst, d, h: M.tab((_basis(src, dst, d) * (2.0 / h if d else 1.0)).T)  # noqa: E731
    # J: (J, chi) = (B, curl chi), exact rules
    bx, by, bz = _at(M, F[0], Q, Q) * wq, _at(M, F[1], Q, Q) * wq, _at(M, F[2], Gs, Gs) * wg
    lz = _axy(bx, T(W, Q, 0, M.hx), T(W, Q, 1, M.hy)) - _axy(by, T(W, Q, 1, M.hx), T(W, Q, 0, M.hy))
    lx = -_axy(bz, T(Gs, Gs, 0, M.hx), T(W, Gs, 1, M.hy))
    ly = _axy(bz, T(W, Gs, 1, M.hx), T(Gs, Gs, 0, M.hy))
    sets = [(Gs, W, M.wg, M.ww), (W, Gs, M.ww, M.wg), (W, W, M.ww, M.ww)]
    wide = [(False, True), (True, False), (True, True)]
    Jg = [_assemble(M, t, s[2], s[3], J0) for t, s in zip((lx, ly, lz), sets)]
    Jl = [(M.local(t, *w), s[0], s[1]) for t, w, s in zip(Jg, wide, sets)]
    Jp = [_at(M, t, P, P) for t in Jl]
    # E = -u x B at the nodes + the resistive term by the GLL_p rule; the Lorentz load on the way
    wp = M.tab(np.outer(M.wp, M.wp) * J0)
    load, Eg = [0.0, 0.0, 0.0], []
    for c, s in enumerate(sets):
        a, b = (c + 1) % 3, (c + 2) % 3
        Bn = [_at(M, F[k], s[0], s[1]) for k in range(3)]
        un = [_at(M, (u[k], P, P), s[0], s[1]) for k in range(3)]
        w = M.tab(np.outer(s[3], s[2]) * J0)
        E = -w * (un[a] * Bn[b] - un[b] * Bn[a])
        if eta is not None:
            E = E + _axy(eta[..., None, None] * wp * Jp[c], T(s[0], P, 0, M.hx), T(s[1], P, 0, M.hy))
        Eg.append(_assemble(M, E, s[2], s[3], J0))
        for k, f in ((a, -Bn[b]), (b, Bn[a])):  # J x B of the component c
            load[k] = load[k] + _axy(w * f * Jl[c][0], T(P, s[0], 0, M.hx), T(P, s[1], 0, M.hy))
    El = [(M.local(t, *w), s[0], s[1]) for t, w, s in zip(Eg, wide, sets)]
    dBx = M.to_grid(-_at(M, El[2], W, Gs, 0, 1))
    dBy = M.to_grid(_at(M, El[2], Gs, W, 1, 0))
    dBz = M.to_grid(_at(M, El[0], M.xv, M.xv, 0, 1) - _at(M, El[1], M.xv, M.xv, 1, 0))
    du = torch.stack(load) / (rho * wp)
    de = torch.zeros_like(rho) if eta is None else eta[..., None, None] * (Jp[0] ** 2 + Jp[1] ** 2 + Jp[2] ** 2) / rho
    return de, du, dBx, dBy, dBz


def _wave(M, rho, u, F, d):
    b = sum(_at(M, f, M.xp, M.xp) ** 2 for f in F)
    return (u[d].abs() + torch.sqrt(b / rho)).amax((-1, -2))


def _resistivity(M, rho, u, B):
    F, amp = _fields(M, B), []
    M1 = M.m + 1
    for k, f in enumerate(F):
        g = B[k][:M.by * M1 + (1 if M.walls & 2 and k == 1 else 0), :M.bx * M1 + (1 if M.walls & 1 and k == 0 else 0)]
        q = _at(M, f, M.xq, M.xq) * M.tab(np.outer(M.wq, M.wq) / 4.0)
        mean = q[:M.by, :M.bx].sum((-1, -2)).mean()
        amp.append(0.0 if bool(g.max() - g.min() <= 1024.0 * EPS * g.abs().max()) else float((g - mean).abs().max()))
    best = torch.zeros(M.ny, M.nx, dtype=torch.float64, device=DEV)
    for d, h in ((0, M.hx), (1, M.hy)):
        shared, sig = max(amp[1 - d], amp[2]), torch.zeros_like(best)
        for k in (1 - d, 2):
            if amp[k] == 0.0:
                continue
            ends = np.array([-1.0, 1.0])
            v = _at(M, F[k], ends, M.xq).transpose(-1, -2) if d == 0 else _at(M, F[k], M.xq, ends)
            jump = v[..., 0, :] - torch.roll(v[..., 1, :], 1, 1 - d)
            s = torch.sqrt((0.5 * M.tab(M.wq) * jump * jump).sum(-1))
            sig = torch.maximum(sig, (s + torch.roll(s, -1, 1 - d)) / (2.0 * shared))
        best = torch.maximum(best, h / (2 * M.p + 1) * _wave(M, rho, u, F, d) * (5.0 * sig).clamp(max=1.0))
    return 0.2 * best


def _shell_basis(M, rho):
    """Values at the nodes of a basis orthonormal under rho times the GLL rule, shell by shell."""
    V, n = npleg.legvander(M.xp, M.p), M.np
    order = sorted(((a, b) for a in range(n) for b in range(n)), key=lambda t: max(t))
    Phi = M.tab(np.stack([np.outer(V[:, b], V[:, a]).reshape(-1) for a, b in order], 1))  # [node][mode]
    W = (rho * M.tab(np.outer(M.wp, M.wp) * M.hx * M.hy / 4.0)).reshape(M.K, -1)
    psi = torch.empty(M.K, n * n, n * n, dtype=torch.float64, device=DEV)
    for at in range(0, M.K, 1 << 16):
        part = W[at:at + (1 << 16)]
        # Gram-Schmidt, twice, in the order of the shells
        A = Phi.expand(len(part), -1, -1).clone()
        for k in range(n * n):
            v = A[..., k]
            for _ in range(2 if k else 0):
                v = v - ((A[..., :k] * (part * v)[..., None]).sum(1)[:, None, :] * A[..., :k]).sum(-1)
            A[..., k] = v / torch.sqrt((part * v * v).sum(1))[:, None]
        psi[at:at + (1 << 16)] = A
    return psi, W, [max(t) for t in order]


def _velocity_oe(M, basis, rho, e, u, B, tau):
    F = _fields(M, B)
    lam = [(2 * M.p + 1) / h * _wave(M, rho, u, F, d) for d, h in ((0, M.hx), (1, M.hy))]
    D = [t.reshape(M.K, 1) for t in _damping(M, _sensor(M, list(u)), lam, 0.02 * tau)]
    psi, W, shell = basis
    heat, new = torch.zeros_like(W), []
    for d in range(3):
        y = ((W * u[d].reshape(M.K, -1))[..., None] * psi).sum(1)
        v = torch.zeros_like(W)
        for l in range(M.np):
            at = [k for k, s in enumerate(shell) if s == l]
            w = sum(psi[..., k] * y[:, k, None] for k in at)
            v = v + D[l] * w
            heat = heat + 0.5 * (1.0 - D[l] ** 2) * w * w
        new.append(v.reshape(u[d].shape))
    return e + heat.reshape(e.shape), torch.stack(new)


def _magnetic(M, case, rho, e, u, B, tau):
    eta = _resistivity(M, rho, u, B) if case["stab"] == "full" else None
    basis = _shell_basis(M, rho) if case["stab"] != "none" else None
    Yn = [e, u, *B]

    def stage(a, b, Y):
        L = _rhs_magnetic(M, rho, Y[1], Y[2:], eta)
        Y = [a * n + b * (s + tau * t) for n, s, t in zip(Yn, Y, L)]
        if basis:
            Y[0], Y[1] = _velocity_oe(M, basis, rho, Y[0], Y[1], Y[2:], tau)
        return Y

    Y = stage(0.0, 1.0, Yn)
    Y = stage(0.75, 0.25, Y)
    Y = stage(1.0 / 3.0, 2.0 / 3.0, Y)
    return Y[0], Y[1], Y[2:]


def _cfl(M, U, B):
    F = _fields(M, B)
    cf = torch.sqrt((GAMMA * _pressure(U) + sum(_at(M, f, M.xp, M.xp) ** 2 for f in F)) / U[0])
    rate = ((U[1] / U[0]).abs() + cf) / M.hx + ((U[2] / U[0]).abs() + cf) / M.hy
    return CFL / ((2 * M.p + 1) * float(rate.max()))


def _primitive(U):
    u = U[1:4] / U[0]
    return U[0], U[4] / U[0] - 0.5 * (u * u).sum(0), u


def _step(M, case, U, B, dt):
    def hydro(tau):
        nonlocal U
        U = _hydro(M, case, U, tau)

    def magnetic(tau):
        nonlocal U, B
        rho, e, u = _primitive(U)
        e, u, B = _magnetic(M, case, rho, e, u, B, tau)
        U = torch.cat([rho[None], rho * u, (rho * e + 0.5 * rho * (u * u).sum(0))[None]])

    inner, outer = (hydro, magnetic) if case["order"] else (magnetic, hydro)
    outer(0.5 * dt)
    inner(dt)
    outer(0.5 * dt)
    return U, B


def exact(case, seed):
    if case["kind"] == "ensemble":
        if case["runs"] > 16:  # over 20 seconds
            return None
        each = [exact(c, seed + 1000 * i) for i, c in enumerate(_members(case))]
        return [torch.cat([r[k].reshape(-1) for r in each]) for k in range(4)]
    M, U, *B = _initial(case, seed)
    shape, V = U.shape, U.reshape(5, M.ny, M.nx, M.np, M.np)
    if case["kind"] == "adjoint":
        eta, cot, cots = _cotangents(case, seed, M, U, B[0])
        el = lambda t: t.reshape(*t.shape[:-3], M.ny, M.nx, M.np, M.np)  # noqa: E731
        grad = _rhs_hydro_vjp(M, V, el(cot)).reshape(shape)
        rho, _, u = _primitive(V)
        leaf = [t.contiguous().requires_grad_() for t in (u, *B)]
        out = _rhs_magnetic(M, rho, leaf[0], leaf[1:], eta.reshape(M.ny, M.nx))
        grads = torch.autograd.grad(out, leaf, [el(cots[0]), el(cots[1]), *cots[2:]])
        flat = lambda t: t.detach().reshape(*t.shape[:-4], M.K, M.np, M.np)  # noqa: E731
        return [_rhs_hydro(M, V).reshape(shape), grad, flat(out[0]), flat(out[1]), *(t.detach() for t in out[2:]), flat(grads[0]), *grads[1:]]
    dt = _cfl(M, V, B)
    if case["kind"] == "hydro":
        return [_hydro(M, case, V, 0.5 * dt).reshape(shape)]
    if case["kind"] == "magnetic":
        e, u, B = _magnetic(M, case, *_primitive(V), B, dt)
        return [e.reshape(shape[1:]), u.reshape(3, *shape[1:]), *B]
    V, B = _step(M, case, V, B, dt)
    return [V.reshape(shape), *B, dt]
