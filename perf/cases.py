"""Workloads by which the speed of this library is judged, each one a call
that a user's program makes through paper_2006_15698_amd.dg.

    listed()             the fixed cases, smallest to largest
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs and solver handle, on the GPU
    run(state)           one pass; returns every output whole
    work(case)           bytes and floating-point operations of one pass
    exact(case, seed)    the outputs by plain torch in 64 bits

Every kind of pass ("path"):
    step      nsteps LSERK45 steps of one mesh in place (Solver.step)
    monitor   one step at the CFL time step of the current state, then the
              conserved integrals: a program that adapts dt and logs
    autograd  the right-hand side and its vector-Jacobian product (RHS)
    gradient  gradient of the kinetic energy through nsteps checkpointed
              steps (rk_gradient)
    hp        steps with a degree per element, a fraction of the cells
              refined once (VariableDegree)
    batch     graph-replayed steps of many meshes of uneven size and degree
              (Batch)
and, for the paths of one mesh, the form of the scheme: euler, fp32 (matrix
core contractions), viscous (Navier-Stokes, Re 1600) and kep (split form).

States are the Taylor-Green vortex at Mach 0.1 on [0, 2 pi]^3 with seeded
smooth perturbations of every primitive variable (density waves on [0, 1]^3
for "wave"), the time step is that of CFL 0.3.
"""

import math

import numpy as np
import torch

from paper_2006_15698_amd import dg

GAMMA = 1.4
CFL = 0.3
MU, PRANDTL = 1.0 / 1600.0, 0.71
TGV_SPEED = 11.0      # |u| + c at Mach 0.1 with V0 = 1
WAVE_SPEED = 3.0      # |u| + c of the density wave (u = 1, p = 1, rho >= 0.7)
FORMS = ("euler", "fp32", "viscous", "kep")


def listed():
    return [
        # the smallest call: the density-wave mesh, one step at a time
        dict(name="wave_4_p1", path="step", form="euler", nx=4, ny=4, nz=4, p=1, nsteps=1, flow="wave"),
        # a small box with unequal odd sides, dt adapted and integrals logged at every step
        dict(name="monitor_13x9x21_p2", path="monitor", form="euler", nx=13, ny=9, nz=21, p=2, nsteps=1, flow="tgv"),
        # gradient of an objective through time stepping, checkpointed
        dict(name="gradient_16_p3", path="gradient", form="euler", nx=16, ny=16, nz=16, p=3, nsteps=8, every=4,
             flow="tgv"),
        # the matrix-core form on a mesh of ordinary size
        dict(name="tgv_24_p5_fp32", path="step", form="fp32", nx=24, ny=24, nz=24, p=5, nsteps=4, flow="tgv"),
        # right-hand side and its adjoint as a layer of a differentiable program
        dict(name="autograd_32_p3", path="autograd", form="euler", nx=32, ny=32, nz=32, p=3, nsteps=1, flow="tgv"),
        # ordinary size, many steps: streams mostly from the last-level cache
        dict(name="tgv_32_p3", path="step", form="euler", nx=32, ny=32, nz=32, p=3, nsteps=10, flow="tgv"),
        # independent small meshes advanced together (parameter studies)
        dict(name="batch_64", path="batch", count=64, nmin=6, nmax=24, pmin=1, pmax=5, nsteps=2, mesh_seed=15698),
        # hp mesh: degrees 3..5, 7.8% of the cells refined
        dict(name="hp_40_p3to5", path="hp", nx=40, ny=40, nz=40, pmin=3, pmax=5, refine=0.7, nsteps=2, mesh_seed=-1),
        # one GPU's share at the paper's per-GPU size, the benchmark's flow, in its three formulations
        dict(name="tgv_48_p4", path="step", form="euler", nx=48, ny=48, nz=48, p=4, nsteps=5, flow="tgv"),
        dict(name="tgv_48_p4_kep", path="step", form="kep", nx=48, ny=48, nz=48, p=4, nsteps=2, flow="tgv"),
        dict(name="tgv_48_p4_re1600", path="step", form="viscous", nx=48, ny=48, nz=48, p=4, nsteps=2, flow="tgv"),
        # the paper's degree
        dict(name="tgv_40_p6", path="step", form="euler", nx=40, ny=40, nz=40, p=6, nsteps=3, flow="tgv"),
    ]


# node-stages that a drawn pass may take, below the largest listed one's
_MAX_NODE_STAGES = 1.5e8


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["step"] * 6 + ["monitor", "monitor", "autograd", "autograd", "gradient", "hp", "hp", "batch"])
    if path == "batch":
        return dict(path=path, count=_log_int(rng, 4, 64), nmin=6, nmax=rng.randint(12, 24), pmin=rng.randint(1, 3),
                    pmax=rng.randint(3, 5), nsteps=rng.randint(1, 3), mesh_seed=rng.randrange(1 << 30))
    if path == "hp":
        pmin = rng.randint(1, 4)
        return dict(path=path, nx=rng.randint(6, 28), ny=rng.randint(6, 28), nz=rng.randint(6, 28), pmin=pmin,
                    pmax=pmin + rng.randint(0, 2), refine=rng.choice([2.0, 0.05, 0.2]), nsteps=rng.randint(1, 3),
                    mesh_seed=rng.randrange(1 << 30))
    form = rng.choice(FORMS + ("euler", "euler")) if path in ("step", "monitor") else "euler"
    p = rng.randint(1, 7)
    limit = 5e4 if path == "gradient" else 3e6 if form in ("viscous", "kep") else 1e7
    top = min(48, int((limit / (p + 1) ** 3) ** (1.0 / 3.0)))
    n = _log_int(rng, 4, max(4, top))
    sides = [min(48, max(3, int(round(n * rng.uniform(0.75, 1.3))))) for _ in range(3)]
    case = dict(path=path, form=form, nx=sides[0], ny=sides[1], nz=sides[2], p=p, nsteps=1,
                flow="wave" if form == "euler" and path == "step" and rng.random() < 0.2 else "tgv")
    if path == "step":
        nodes = sides[0] * sides[1] * sides[2] * (p + 1) ** 3
        case["nsteps"] = max(1, min(rng.choice([1, 2, 3, 5, 10]), int(_MAX_NODE_STAGES / (5 * nodes))))
    if path == "gradient":
        case["nsteps"] = rng.randint(3, 8)
        case["every"] = rng.randint(2, 5)
    return case


# ---- meshes and states -------------------------------------------------------
def _lengths(flow):
    return (1.0,) * 3 if flow == "wave" else (2.0 * math.pi,) * 3


def _gauss(N):
    return np.polynomial.legendre.leggauss(N)


class _Flow:
    """The seeded primitive fields, as functions of position."""

    def __init__(self, flow, seed):
        self.flow = flow
        rng = np.random.default_rng([seed, 15698])
        # wave: amplitude; tgv: four smooth modes for each of rho, u, v, w, p
        self.amp = rng.uniform(0.1, 0.3)
        self.k = rng.integers(-2, 3, size=(5, 4, 3))
        self.phase = rng.uniform(0.0, 2.0 * math.pi, size=(5, 4))
        self.a = rng.uniform(-1.0, 1.0, size=(5, 4)) * 2.5e-3

    def conserved(self, x, y, z):
        if self.flow == "wave":
            rho = 1.0 + self.amp * torch.sin(2.0 * math.pi * (x + y + z) + float(self.phase[0, 0]))
            u, v, w = torch.ones_like(rho), torch.ones_like(rho), torch.ones_like(rho)
            p = torch.ones_like(rho)
        else:
            def bump(f):
                return sum(float(self.a[f, m]) * torch.sin(int(self.k[f, m, 0]) * x + int(self.k[f, m, 1]) * y
                                                           + int(self.k[f, m, 2]) * z + float(self.phase[f, m]))
                           for m in range(4))
            p0 = 100.0 / GAMMA
            p = p0 + (torch.cos(2 * x) + torch.cos(2 * y)) * (torch.cos(2 * z) + 2.0) / 16.0
            rho = p / p0 * (1.0 + bump(0))
            u = torch.sin(x) * torch.cos(y) * torch.cos(z) + bump(1)
            v = -torch.cos(x) * torch.sin(y) * torch.cos(z) + bump(2)
            w = torch.zeros_like(rho) + bump(3)
            p = p * (1.0 + bump(4))
        return torch.stack([rho, rho * u, rho * v, rho * w, p / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v + w * w)])


def _box_state(n, p, L, flow, device):
    """State [5, nz, ny, nx, N, N, N] of a uniform mesh."""
    x1, _ = _gauss(p + 1)
    axes = []
    for d in range(3):
        h = L[d] / n[d]
        c = (np.arange(n[d])[:, None] * h + (x1[None, :] + 1.0) * (h / 2.0))
        shape = [1] * 6
        shape[2 - d], shape[5 - d] = n[d], p + 1
        axes.append(torch.from_numpy(c).to(device).reshape(shape))
    full = (n[2], n[1], n[0], p + 1, p + 1, p + 1)
    return flow.conserved(*(a.expand(full) for a in axes)).contiguous()


def _box_dt(n, p, L, speed):
    return CFL / ((2 * p + 1) * speed * sum(m / l for m, l in zip(n, L)))


def _batch_specs(case):
    rng = np.random.default_rng(case["mesh_seed"])
    out = []
    for i in range(case["count"]):
        out.append((int(rng.integers(case["nmin"], case["nmax"] + 1)), int(rng.integers(case["pmin"], case["pmax"] + 1)),
                    "wave" if rng.integers(0, 2) else "tgv"))
    return out


class _HpMesh:
    """Cells, elements and degrees of an hp case.  Positions and sizes are in
    units of half a cell; elements cell by cell, a refined cell's children
    (kz, ky, kx)."""

    def __init__(self, case):
        nx, ny, nz = self.n = (case["nx"], case["ny"], case["nz"])
        self.L = _lengths("tgv")
        cz, cy, cx = (a.reshape(-1) for a in np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij"))
        span = case["pmax"] - case["pmin"]
        if case["mesh_seed"] < 0:
            # an hp indicator's choice: the vortex's initial enstrophy density
            X, Y, Z = ((c + 0.5) * (2.0 * math.pi / m) for c, m in ((cx, nx), (cy, ny), (cz, nz)))
            ind = np.sqrt((np.cos(X) * np.sin(Y) * np.sin(Z)) ** 2 + (np.sin(X) * np.cos(Y) * np.sin(Z)) ** 2
                          + (2 * np.sin(X) * np.sin(Y) * np.cos(Z)) ** 2) / 2.0
            refine = (ind >= case["refine"]).astype(np.int64)
            deg = case["pmin"] + np.rint(span * ind).astype(np.int64)
        else:
            # seeded; a "refine" above 1 leaves every cell whole
            rng = np.random.default_rng(case["mesh_seed"])
            refine = (rng.random(cx.size) < (case["refine"] if case["refine"] < 1 else 0.0)).astype(np.int64)
            deg = rng.integers(case["pmin"], case["pmax"] + 1, size=cx.size)
        self.refine = refine
        count = np.where(refine == 1, 8, 1)
        cell = np.repeat(np.arange(cx.size), count)
        rank = np.arange(cell.size) - np.repeat(np.cumsum(count) - count, count)
        self.size = np.where(refine[cell] == 1, 1, 2)
        kid = np.stack([rank % 2, (rank // 2) % 2, rank // 4], axis=1)
        self.pos = 2 * np.stack([cx, cy, cz], axis=1)[cell] + np.where(self.size[:, None] == 1, kid, 0)
        self.deg = deg[cell]
        self.off = np.concatenate([[0], np.cumsum((self.deg + 1) ** 3)])
        self.T = int(self.off[-1])

    def nodes(self, p, device):
        """Elements of degree p and the index of their nodes, [E_p, N^3]."""
        es = np.flatnonzero(self.deg == p)
        idx = torch.from_numpy(self.off[es]).to(device)[:, None] + torch.arange((p + 1) ** 3, device=device)
        return es, idx

    def state(self, flow, device):
        Q = torch.empty(5, self.T, dtype=torch.float64, device=device)
        half = [l / (2 * m) for l, m in zip(self.L, self.n)]
        for p in np.unique(self.deg):
            N = int(p) + 1
            es, idx = self.nodes(int(p), device)
            x1 = torch.from_numpy(_gauss(N)[0]).to(device)
            size = torch.from_numpy(self.size[es].astype(np.float64)).to(device)[:, None]
            xyz = []
            for d in range(3):
                c = torch.from_numpy(self.pos[es, d].astype(np.float64)).to(device)[:, None] + (x1 + 1.0) * 0.5 * size
                shape = [len(es), 1, 1, 1]
                shape[3 - d] = N
                xyz.append((c * half[d]).reshape(shape).expand(-1, N, N, N).reshape(len(es), -1))
            Q[:, idx] = flow.conserved(*xyz)
        return Q.reshape(-1)

    def dt(self):
        fine = 2 if self.refine.any() else 1
        return _box_dt([fine * m for m in self.n], int(self.deg.max()), self.L, TGV_SPEED)


def _box(case):
    return (case["nx"], case["ny"], case["nz"])


def _dt(case):
    n, p, L = _box(case), case["p"], _lengths(case["flow"])
    dt = _box_dt(n, p, L, WAVE_SPEED if case["flow"] == "wave" else TGV_SPEED)
    if case["form"] == "viscous":
        nu = MU * GAMMA / PRANDTL
        dt = 1.0 / (1.0 / dt + (2 * p + 1) ** 2 * nu * sum((m / l) ** 2 for m, l in zip(n, L)) / CFL)
    return dt


def prepare(case, seed):
    dev = torch.device("cuda")
    path = case["path"]
    if path == "batch":
        specs = _batch_specs(case)
        ns, ps, Ls = [(n,) * 3 for n, _, _ in specs], [p for _, p, _ in specs], [_lengths(f) for _, _, f in specs]
        b = dg.Batch(ns, ps, Ls)
        Q = b.empty()
        for i, (n, p, f) in enumerate(specs):
            b.view(Q, i).copy_(_box_state(ns[i], p, Ls[i], _Flow(f, seed * 1009 + i), dev))
        b.set_dt([_box_dt(ns[i], ps[i], Ls[i], WAVE_SPEED if f == "wave" else TGV_SPEED)
                  for i, (_, _, f) in enumerate(specs)])
        return dict(case=case, solver=b, Q=Q, res=torch.zeros_like(Q))
    if path == "hp":
        mesh = _HpMesh(case)
        refined = bool(mesh.refine.any())
        v = dg.VariableDegree(mesh.n, mesh.deg, L=mesh.L, refine=mesh.refine if refined else None)
        Q = mesh.state(_Flow("tgv", seed), dev)
        return dict(case=case, solver=v, Q=Q, res=torch.zeros_like(Q), dt=mesh.dt())
    form, L = case["form"], _lengths(case["flow"])
    s = dg.Solver(_box(case), case["p"], L=L, precision=dg.DG_FP32_MFMA if form == "fp32" else dg.DG_FP64,
                  mu=MU if form == "viscous" else 0.0, prandtl=PRANDTL,
                  volume_form=dg.DG_VOLUME_KEP if form == "kep" else dg.DG_VOLUME_STANDARD)
    Q = _box_state(_box(case), case["p"], L, _Flow(case["flow"], seed), dev)
    st = dict(case=case, solver=s, Q=Q, res=torch.zeros_like(Q), dt=_dt(case))
    if path == "autograd":
        st["Q"] = Q.requires_grad_(True)
        st["gR"] = _cotangent(Q, seed)
    return st


def _cotangent(Q, seed):
    """Seeded weights of the rates, each field scaled by the field's size."""
    g = torch.Generator(device="cpu").manual_seed(seed)
    w = torch.randn(Q.shape, dtype=torch.float64, generator=g).to(Q.device)
    with torch.no_grad():
        return w / Q.abs().amax(dim=tuple(range(1, Q.dim())), keepdim=True)


def run(state):
    case, s, Q, res = state["case"], state["solver"], state["Q"], state["res"]
    path = case["path"]
    if path == "step" or path == "hp":
        s.step(Q, res, state["dt"], case["nsteps"])
        return Q, res
    if path == "batch":
        s.step(Q, res, nsteps=case["nsteps"], graph=True)
        return Q, res
    if path == "monitor":
        dt = s.dt_cfl(Q, CFL)
        s.step(Q, res, dt)
        return Q, res, dt, s.integrals(Q)
    if path == "autograd":
        R = dg.RHS.apply(Q, s)
        (gQ,) = torch.autograd.grad(R, Q, state["gR"])
        return R.detach(), gQ
    return dg.rk_gradient(s, Q, state["dt"], case["nsteps"], dg.kinetic_energy_grad(s), every=case["every"])


# ---- the work of one pass ------------------------------------------------------
def _stage_flops(N, form="euler"):
    """Per node and stage: fluxes and volume contraction 38 + 30 N, surface
    3 (40 N + 76) / N, inverse mass and update 30.  The split form evaluates
    a two-point flux per pair of nodes of a line instead of a flux per node;
    the viscous terms add the gradients of four quantities, the viscous flux
    and its derivative."""
    base = 38 + 30 * N + 3 * (40 * N + 76) / N + 30
    if form == "kep":
        return base + 3 * (13 * (N + 1) / 2 + 5 * N)
    if form == "viscous":
        return base + 3 * 2 * (8 * N + 40) + 80
    return base


def work(case):
    """A stage reads the state and the residual and writes both, 160 bytes a
    node (the first stage of a step reads no residual: 120)."""
    path = case["path"]
    step = 120 + 4 * 160
    if path == "batch":
        sizes = [(n ** 3 * (p + 1) ** 3, p + 1) for n, p, _ in _batch_specs(case)]
        return dict(bytes=case["nsteps"] * step * sum(m for m, _ in sizes),
                    flops=5 * case["nsteps"] * sum(m * _stage_flops(N) for m, N in sizes))
    if path == "hp":
        mesh = _HpMesh(case)
        per = (mesh.deg + 1) ** 3
        return dict(bytes=case["nsteps"] * step * mesh.T,
                    flops=5 * case["nsteps"] * float(sum(int(per[mesh.deg == p].sum()) * _stage_flops(int(p) + 1)
                                                         for p in np.unique(mesh.deg))))
    N = case["p"] + 1
    nodes = case["nx"] * case["ny"] * case["nz"] * N ** 3
    flops = nodes * _stage_flops(N, case["form"])
    if path == "step":
        return dict(bytes=case["nsteps"] * step * nodes, flops=5 * case["nsteps"] * flops)
    if path == "monitor":   # the wave speed and the integrals read the state once more each
        return dict(bytes=(step + 80) * nodes, flops=5 * flops + 60 * nodes)
    if path == "autograd":  # rate: state in, rate out; adjoint: state and weights in, gradient out
        return dict(bytes=200 * nodes, flops=3 * flops)
    # gradient: forward, recomputation, and five reverse stages a step (state
    # and two adjoints in, two adjoints out), one checkpoint written and read
    # per segment
    segments = -(-case["nsteps"] // case["every"])
    return dict(bytes=nodes * (case["nsteps"] * (2 * step + 5 * 200) + segments * 80 + 80),
                flops=flops * 5 * case["nsteps"] * 4)


# ---- the same outputs by plain torch in 64 bits --------------------------------
_RKA = (0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
        -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0)
_RKB = (1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0, 1720146321549.0 / 2090206949498.0,
        3134564353537.0 / 4481467310338.0, 2277821191437.0 / 14882151754819.0)


def _gauss_long(N):
    """Gauss-Legendre rule in extended precision: Newton steps on P_N."""
    x = np.polynomial.legendre.leggauss(N)[0].astype(np.longdouble)
    for _ in range(3):
        p0, p1 = np.ones_like(x), x
        for k in range(2, N + 1):
            p0, p1 = p1, ((2 * k - 1) * x * p1 - (k - 1) * p0) / k
        dp = N * (x * p1 - p0) / (x * x - 1)
        x = x - p1 / dp
    return x, 2 / ((1 - x * x) * dp * dp)


def _lagrange(nodes, x):
    """l_a(x_i), shaped [len(x), len(nodes)]."""
    x = np.atleast_1d(np.asarray(x, dtype=np.longdouble))
    out = np.ones((len(x), len(nodes)), dtype=np.longdouble)
    for a in range(len(nodes)):
        for m in range(len(nodes)):
            if m != a:
                out[:, a] *= (x - nodes[m]) / (nodes[a] - nodes[m])
    return out


def _derivative(nodes):
    """D[i, a] = l_a'(x_i)."""
    N = len(nodes)
    D = np.zeros((N, N), dtype=np.longdouble)
    for a in range(N):
        for i in range(N):
            for m in range(N):
                if m != a:
                    t = 1 / (nodes[a] - nodes[m])
                    for q in range(N):
                        if q != a and q != m:
                            t *= (nodes[i] - nodes[q]) / (nodes[a] - nodes[q])
                    D[i, a] += t
    return D


class _Line:
    """Operators of one line of N Gauss-Legendre nodes."""

    def __init__(self, N, device):
        x, w = _gauss_long(N)

        def up(a):
            return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(device)
        self.N, self.x, self.w = N, x, w
        D = _derivative(x)
        self.D = up(D)
        self.Dh = up((w[:, None] * D).T / w[:, None])        # w_a l_i'(x_a) / w_i
        ends = _lagrange(x, [-1, 1])
        self.lm, self.lp = up(ends[0]), up(ends[1])
        self.lift_m, self.lift_p = up(ends[0] / w), up(ends[1] / w)


def _along(A, X, axis):
    """sum_a A[i, a] X[..., a, ...] along a node axis."""
    return torch.movedim(torch.movedim(X, axis, -1) @ A.T, -1, axis)


def _trace(l, X, axis):
    return torch.movedim(X, axis, -1) @ l


def _lift(l, F, axis):
    return torch.movedim(F.unsqueeze(-1) * l, -1, axis)


def _pressure(q):
    return (GAMMA - 1.0) * (q[4] - 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / q[0])


def _flux(q, d):
    p = _pressure(q)
    ud = q[1 + d] / q[0]
    return torch.stack([q[1 + d]] + [q[1 + k] * ud + (p if k == d else 0.0) for k in range(3)] + [(q[4] + p) * ud])


def _lax_friedrichs(a, b, d):
    la = (a[1 + d] / a[0]).abs() + torch.sqrt(GAMMA * _pressure(a) / a[0])
    lb = (b[1 + d] / b[0]).abs() + torch.sqrt(GAMMA * _pressure(b) / b[0])
    return 0.5 * (_flux(a, d) + _flux(b, d)) - 0.5 * torch.where(la >= lb, la, lb) * (b - a)


def _two_point(a, b, d):
    """Kennedy-Gruber flux between primitive states (rho, u, v, w, p, e)."""
    mean = [0.5 * (s + t) for s, t in zip(a, b)]
    m = mean[0] * mean[1 + d]
    return torch.stack([m] + [m * mean[1 + k] + (mean[4] if k == d else 0.0) for k in range(3)]
                       + [m * mean[5] + mean[4] * mean[1 + d]])


def _primitives(q):
    return [q[0], q[1] / q[0], q[2] / q[0], q[3] / q[0], _pressure(q), q[4] / q[0]]


def _weak(ln, X, d, sc):
    """Weak derivative along d with the mean of both traces on the faces."""
    node, elem = -1 - d, X.dim() - 4 - d
    mean = 0.5 * (_trace(ln.lp, X, node) + torch.roll(_trace(ln.lm, X, node), -1, elem))
    return sc * (_lift(ln.lift_p, mean, node) - _lift(ln.lift_m, torch.roll(mean, 1, elem), node)
                 - _along(ln.Dh, X, node))


def _viscous_rate(ln, q, sc):
    rho, u, v, w, p, _ = _primitives(q)
    vel = (u, v, w)
    P = torch.stack([u, v, w, p / rho])
    g = [_weak(ln, P, d, sc[d]) for d in range(3)]
    kappa = MU * (GAMMA / (GAMMA - 1.0)) / PRANDTL
    div = g[0][0] + g[1][1] + g[2][2]
    out = torch.zeros_like(q)
    for d in range(3):
        tau = [MU * (g[d][k] + g[k][d]) - ((2.0 / 3.0) * MU * div if k == d else 0.0) for k in range(3)]
        F = torch.stack(tau + [kappa * g[d][3] + sum(vel[k] * tau[k] for k in range(3))])
        out[1:] += _weak(ln, F, d, sc[d])
    return out


def _box_rate(ln, q, sc, form):
    """dQ/dt of a uniform mesh, q [5, nz, ny, nx, N, N, N]."""
    out = torch.zeros_like(q)
    for d in range(3):
        node, elem = -1 - d, 3 - d
        tm, tp = _trace(ln.lm, q, node), _trace(ln.lp, q, node)
        right = _lax_friedrichs(tp, torch.roll(tm, -1, elem), d)
        left = torch.roll(right, 1, elem)
        if form == "kep":
            node_of = [[f.unbind(node) for f in _primitives(q)]]
            line = [[node_of[0][f][i] for f in range(6)] for i in range(ln.N)]
            rows = []
            for (t, F, l) in ((tm, left, ln.lm), (tp, right, ln.lp)):
                e = _primitives(t)
                G = F - sum(l[a] * _two_point(e, line[a], d) for a in range(ln.N))
                rows.append((e, G, l))
            R = []
            for i in range(ln.N):
                pair = [_two_point(line[i], line[a], d) for a in range(ln.N)]
                r = sum(2.0 * ln.D[i, a] * pair[a] for a in range(ln.N))
                for sign, lift, (e, G, l) in ((-1.0, ln.lift_m, rows[0]), (1.0, ln.lift_p, rows[1])):
                    B = _two_point(line[i], e, d) - sum(l[a] * pair[a] for a in range(ln.N)) + G
                    r = r + sign * lift[i] * B
                R.append(-r)
            out = out + sc[d] * torch.stack(R, dim=node)
        else:
            out = out + sc[d] * (_along(ln.Dh, _flux(q, d), node) + _lift(ln.lift_m, left, node)
                                 - _lift(ln.lift_p, right, node))
    if form == "viscous":
        out = out + _viscous_rate(ln, q, sc)
    return out


class _HpRate:
    """dQ/dt of an hp mesh: every face integrated on the Gauss-Legendre rule
    of the higher degree, on the smaller of its two faces."""

    def __init__(self, mesh, device):
        self.mesh, self.device = mesh, device
        self.degs = [int(p) for p in np.unique(mesh.deg)]
        self.lines = {p: _Line(p + 1, device) for p in self.degs}
        self.elems = {p: mesh.nodes(p, device) for p in self.degs}
        self.sc = {p: [torch.from_numpy(4.0 * m / (l * mesh.size[es])).to(device) for m, l in zip(mesh.n, mesh.L)]
                   for p, (es, _) in self.elems.items()}
        local = np.zeros(mesh.deg.size, dtype=np.int64)
        for p, (es, _) in self.elems.items():
            local[es] = np.arange(len(es))
        # owner of every half-cell, then every half-cell face between two elements
        fine = [2 * m for m in mesh.n]
        owner = np.zeros((fine[2], fine[1], fine[0]), dtype=np.int64)
        for kz in range(2):
            for ky in range(2):
                for kx in range(2):
                    k = np.minimum(np.array([kx, ky, kz]), mesh.size[:, None] - 1)
                    x, y, z = (mesh.pos + k).T
                    owner[z, y, x] = np.arange(mesh.deg.size)
        self.groups = []
        grid = np.meshgrid(*(np.arange(f) for f in reversed(fine)), indexing="ij")[::-1]
        for d in range(3):
            a, b = owner.reshape(-1), np.roll(owner, -1, axis=2 - d).reshape(-1)
            t = [grid[c].reshape(-1) % 2 for c in range(3) if c != d]
            whole = (mesh.size[a] == 2) & (mesh.size[b] == 2)
            keep = (a != b) & ~(whole & ((t[0] == 1) | (t[1] == 1)))
            a, b, t = a[keep], b[keep], [c[keep] for c in t]
            hang = mesh.size[a] != mesh.size[b]
            side = np.where(hang, np.where(mesh.size[a] == 2, 1, 2), 0)   # which side is the larger
            key = np.stack([mesh.deg[a], mesh.deg[b], side, np.where(hang, t[0], 0), np.where(hang, t[1], 0)], axis=1)
            for row in np.unique(key, axis=0):
                m = (key == row).all(axis=1)
                self.groups.append((d, [int(v) for v in row], torch.from_numpy(local[a[m]]).to(device),
                                    torch.from_numpy(local[b[m]]).to(device)))

    def _maps(self, p, M, quarter):
        """Interpolation to the mortar points and projection back, per
        tangential direction (lower axis first)."""
        ln = self.lines[p]
        xm, wm = _gauss_long(M)
        out = []
        for o in quarter:
            I = _lagrange(ln.x, xm if o is None else (xm + 2 * o - 1) / 2)
            P = (I * wm[:, None]).T / ln.w[:, None] / (1 if o is None else 2)
            out.append(tuple(torch.from_numpy(np.ascontiguousarray(m, dtype=np.float64)).to(self.device)
                             for m in (I, P)))
        return out

    def __call__(self, Qflat):
        Q = Qflat.view(5, -1)
        S, T, G = {}, {}, {}
        for p, (es, idx) in self.elems.items():
            N = p + 1
            S[p] = Q[:, idx].view(5, -1, N, N, N)
            for d in range(3):
                for side, l in ((0, self.lines[p].lm), (1, self.lines[p].lp)):
                    T[p, d, side] = _trace(l, S[p], -1 - d)
                    G[p, d, side] = torch.zeros_like(T[p, d, side])
        for d, (pa, pb, big, t0, t1), a, b in self.groups:
            M = max(pa, pb) + 1
            ma = self._maps(pa, M, (t0, t1) if big == 1 else (None, None))
            mb = self._maps(pb, M, (t0, t1) if big == 2 else (None, None))

            def mortar(t, m):
                return _along(m[1][0], _along(m[0][0], t, -1), -2)

            def project(f, m):
                return _along(m[1][1], _along(m[0][1], f, -1), -2)
            f = _lax_friedrichs(mortar(T[pa, d, 1][:, a], ma), mortar(T[pb, d, 0][:, b], mb), d)
            G[pa, d, 1].index_add_(1, a, project(f, ma))
            G[pb, d, 0].index_add_(1, b, project(f, mb))
        out = torch.empty_like(Q)
        for p, (es, idx) in self.elems.items():
            ln = self.lines[p]
            r = 0.0
            for d in range(3):
                node = -1 - d
                r = r + self.sc[p][d].view(-1, 1, 1, 1) * (_along(ln.Dh, _flux(S[p], d), node)
                                                           + _lift(ln.lift_m, G[p, d, 0], node)
                                                           - _lift(ln.lift_p, G[p, d, 1], node))
            out[:, idx] = r.reshape(5, len(es), -1)
        return out.reshape(-1)


def _integrate(rate, Q, dt, nsteps):
    res = torch.zeros_like(Q)
    for _ in range(nsteps):
        for a, b in zip(_RKA, _RKB):
            res = a * res + dt * rate(Q)
            Q = Q + b * res
    return Q, res


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    path = case["path"]
    if path == "hp":
        mesh = _HpMesh(case)
        return _integrate(_HpRate(mesh, dev), mesh.state(_Flow("tgv", seed), dev), mesh.dt(), case["nsteps"])
    if path == "batch":
        outs = []
        for i, (m, p, f) in enumerate(_batch_specs(case)):
            n, L = (m,) * 3, _lengths(f)
            ln, sc = _Line(p + 1, dev), [2.0 * m / l for l in L]
            outs.append(_integrate(lambda q: _box_rate(ln, q, sc, "euler"),
                                   _box_state(n, p, L, _Flow(f, seed * 1009 + i), dev),
                                   _box_dt(n, p, L, WAVE_SPEED if f == "wave" else TGV_SPEED), case["nsteps"]))
        return tuple(torch.cat([o[k].reshape(-1) for o in outs]) for k in range(2))
    n, p, L, form = _box(case), case["p"], _lengths(case["flow"]), case["form"]
    ln, sc = _Line(p + 1, dev), [2.0 * m / l for m, l in zip(n, L)]
    Q = _box_state(n, p, L, _Flow(case["flow"], seed), dev)

    def rate(q):
        return _box_rate(ln, q, sc, form)
    if path == "step":
        return _integrate(rate, Q, _dt(case), case["nsteps"])
    w = torch.from_numpy(ln.w.astype(np.float64)).to(dev)
    Jw = (w[:, None, None] * w[None, :, None] * w[None, None, :]) / (sc[0] * sc[1] * sc[2])
    if path == "monitor":
        c = torch.sqrt(GAMMA * _pressure(Q) / Q[0])
        speed = sum(((Q[1 + d] / Q[0]).abs() + c) * (sc[d] / 2.0) for d in range(3)).max()
        dt = float(CFL / ((2 * p + 1) * speed))
        Q, res = _integrate(rate, Q, dt, 1)
        ke = 0.5 * (Q[1] * Q[1] + Q[2] * Q[2] + Q[3] * Q[3]) / Q[0]
        return Q, res, dt, [float((Jw * f).sum()) for f in [*Q, ke]]
    if path == "autograd":
        gR = _cotangent(Q, seed)
        Q.requires_grad_(True)
        R = rate(Q)
        (gQ,) = torch.autograd.grad(R, Q, gR)
        return R.detach(), gQ
    # gradient: forward states kept stage by stage, then the stages reversed
    states, dt = [], _dt(case)
    res = torch.zeros_like(Q)
    for _ in range(case["nsteps"]):
        for a, b in zip(_RKA, _RKB):
            states.append((a, b, Q))
            res = a * res + dt * rate(Q)
            Q = Q + b * res
    u2 = (Q[1] * Q[1] + Q[2] * Q[2] + Q[3] * Q[3]) / (Q[0] * Q[0])
    gQ = torch.stack([-0.5 * u2 * Jw] + [Q[1 + d] / Q[0] * Jw for d in range(3)] + [torch.zeros_like(u2)])
    gres = torch.zeros_like(gQ)
    for a, b, q in reversed(states):
        g = gres + b * gQ
        q = q.detach().requires_grad_(True)
        (v,) = torch.autograd.grad(rate(q), q, g)
        gQ = gQ + dt * v
        gres = a * g
    return gQ, Q
