"""Timed cases of the block-forest finite-volume library and its multigrid solvers.

Every case is work that a program using this library has it do, through the Python entry points
(``forest.GpuForest``, ``multigrid.GpuMultigrid``, ``multigrid.GpuForestMultigrid``, ``mlp.Trainer``):
a few time steps from a given state, a regrid, a solve, a training epoch.  ``prepare`` builds what such
a program already holds (the forest or solver handle, the initial state on the GPU), ``run`` does one
pass, ``work`` counts what the pass cannot do without, and ``exact`` gives the same result in plain
64-bit torch where the discretisation is one that a short program can restate (uniform grids, the
perceptron); the composite operators of refined forests and MHD-HLLC have no such value.
"""
from __future__ import annotations

import functools
import math
import os

import numpy as np
import torch

import workloads as W
from paper_2004_03275_amd import _native as N
from paper_2004_03275_amd import mlp as L
from paper_2004_03275_amd import multigrid as M
from paper_2004_03275_amd.forest import GpuForest, courant_ramp

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(L.__file__)), "data", "flagger_weights.npy")


def listed() -> list:
    return [
        # the smallest call: a 1D shock tube of one block, device-timed steps replayed from a graph
        dict(name="sod_1d", kind="fv", problem="sod", base=1, nx=1024, levels=1, steps=20, arith="exact"),
        # 2D hydrodynamics on 256 uniform leaves in the fast arithmetic, device-timed steps
        dict(name="kh_2d", kind="fv", problem="kh", base=16, levels=1, steps=20, arith="fast"),
        # 2D MHD with GLM cleaning on 1,024 uniform leaves (bit-exact arithmetic, the library's default)
        dict(name="orszag_tang_2d", kind="fv", problem="ot", base=32, levels=1, steps=10, arith="exact"),
        # the paper's circular dam break on a three-level quadtree, host-chosen time steps as a driver
        # script takes them (max_dt, advance)
        dict(name="dam_break_2d_amr", kind="fv", problem="dam", base=6, levels=3, steps=10, arith="exact",
             driver="host"),
        # an adaptive 3D run between two regrids: steps, the learned flagger, the regrid and its transfer
        dict(name="blast_3d_regrid", kind="fv", problem="blast", base=8, levels=3, steps=5, arith="exact",
             flag="mlp", regrid=True),
        # the large run: the 3D AMR blast of 19,384 leaves (79M cells) between two Loehner flaggings
        dict(name="blast_3d_large", kind="fv", problem="blast", base=16, levels=4, steps=5, arith="fast",
             flag="lohner", persistent=True),
        # the paper's 3D MHD blast (HLLC, Cada's limiter), the ramped Courant steps at its start
        dict(name="mhd_blast_3d", kind="fv", problem="mhdblast", base=4, levels=3, steps=5, arith="fast",
             driver="host", variant=2, graph=True),
        # the paper's timed reaction-diffusion step: Schnakenberg 256^2, IMEX through the multigrid solver
        dict(name="rd_2d_imex", kind="rd", ndim=2, n=256, model="schnakenberg", scheme="imex", dt=1e-3, steps=4),
        # the same model in 3D
        dict(name="rd_3d_imex", kind="rd", ndim=3, n=128, model="schnakenberg", scheme="imex", dt=1e-3, steps=2),
        # the paper's Gray-Scott AMR setup: IMEX steps through the forest multigrid
        dict(name="gray_scott_2d_amr", kind="rdf", base=8, levels=3, scheme="imex", dt=0.5, steps=2),
        # a Helmholtz solve on a four-level octree forest (14.5M cells)
        dict(name="helmholtz_3d_amr", kind="helm", ndim=3, base=4, levels=4, radius=0.25, lam=1e4, bc="periodic"),
        # an epoch of the refinement flagger's training in batches of 1,024, the last one partial
        dict(name="flagger_training", kind="train", samples=16000, batch=1024),
    ]


def draw(rng) -> dict:
    """One more case of the same ranges (block counts, grid sizes and batch sizes over their logarithm)."""

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["sod", "kh", "ot", "dam", "blast", "mhdblast", "rd", "rd", "rdf", "helm", "helm", "train"])
    arith = rng.choice(["exact", "fast"])
    if kind == "sod":
        return dict(kind="fv", problem="sod", base=log_int(1, 16), nx=2 * log_int(32, 1024), levels=1,
                    steps=rng.randint(5, 20), arith="exact")
    if kind == "kh":
        return dict(kind="fv", problem="kh", base=log_int(3, 32), levels=1, steps=rng.randint(4, 20), arith=arith)
    if kind == "ot":
        return dict(kind="fv", problem="ot", base=log_int(3, 40), levels=1, steps=rng.randint(4, 12), arith="exact",
                    driver=rng.choice(["host", "device"]))
    if kind == "dam":
        return dict(kind="fv", problem="dam", base=rng.randint(3, 9), levels=rng.randint(2, 4),
                    steps=rng.randint(4, 12), arith=arith, driver=rng.choice(["host", "device"]),
                    flag=rng.choice(["none", "lohner"]))
    if kind == "blast":
        return dict(kind="fv", problem="blast", base=rng.randint(3, 8), levels=rng.randint(2, 3),
                    steps=rng.randint(2, 6), arith=arith, flag=rng.choice(["lohner", "mlp"]),
                    limiter=rng.choice(["vanleer", "vanleer", "koren", "mc"]), regrid=rng.random() < 0.5)
    if kind == "mhdblast":
        return dict(kind="fv", problem="mhdblast", base=rng.randint(3, 5), levels=rng.randint(1, 2),
                    steps=rng.randint(2, 5), arith=arith, driver=rng.choice(["host", "device"]), variant=2,
                    graph=rng.random() < 0.5)
    if kind == "rd":
        nd = rng.choice([2, 2, 3])
        model = rng.choice(["schnakenberg", "gray_scott"])
        return dict(kind="rd", ndim=nd, n=2 ** (rng.randint(5, 10) if nd == 2 else rng.randint(4, 7)), model=model,
                    scheme=rng.choice(["imex", "split", "midpoint"]),
                    dt=(1e-3 if model == "schnakenberg" else 0.5) * rng.uniform(0.5, 1.0), steps=rng.randint(1, 4))
    if kind == "rdf":
        return dict(kind="rdf", base=rng.choice([2, 4, 8]), levels=rng.randint(2, 3),
                    scheme=rng.choice(["imex", "split", "midpoint"]), dt=0.5 * rng.uniform(0.5, 1.0),
                    steps=rng.randint(1, 3))
    if kind == "helm":
        nd = rng.choice([2, 3])
        return dict(kind="helm", ndim=nd, base=rng.choice([2, 4]), levels=rng.randint(2, 4) if nd == 2
                    else rng.randint(1, 3), radius=rng.uniform(0.2, 0.35), lam=10.0 ** rng.uniform(1.0, 4.5),
                    bc=rng.choice(["periodic", "neumann"]))
    return dict(kind="train", samples=log_int(500, 20000), batch=32 * log_int(2, 64))


# ---------------------------------------------------------------------------
# finite-volume cases
# ---------------------------------------------------------------------------

LIMITERS = {"minmod": W.MINMOD, "vanleer": W.VANLEER, "mc": W.MC, "koren": W.KOREN, "cada": W.CADA}


@functools.lru_cache(maxsize=None)
def _fv_forest(problem: str, base: int, nx: int, levels: int, limiter: str):
    """The scheme and leaf list (the same for every seed: a program builds it once)."""
    if problem == "sod":
        s = W.sod_scheme(nx)
        s.base_blocks = (base, 1, 1)
    elif problem == "kh":
        s = W.kh_scheme(base)
    elif problem == "ot":
        s = W.ot_scheme(base)
    elif problem == "dam":
        s = W.dam_break_scheme(base, levels)
    elif problem == "blast":
        s = W.blast_scheme(base, levels)
    else:
        s = W.mhd_blast_scheme(3, base, levels)
    if limiter:
        s.limiter = LIMITERS[limiter]
    if problem in ("sod", "kh", "ot") or levels == 1:
        return W.uniform_forest(s)
    if problem == "blast" and (base, levels) == (16, 4):
        return W.blast_lohner_forest(s)
    radius = {"dam": 2.5, "blast": 0.12, "mhdblast": 0.1}[problem]
    return W.blast_forest(s, radius, buffer_cells=8.0 if problem == "blast" and base == 16 else 4.0)


def _forest(case):
    return _fv_forest(case["problem"], case["base"], case.get("nx", 16), case["levels"], case.get("limiter", ""))


def _centres(f):
    """Cell centres on the GPU, [leaf][z][y][x] per dimension."""
    s, out = f.scheme, []
    lev = torch.from_numpy(f.level.astype(np.int64)).cuda()
    ijk = torch.from_numpy(f.ijk.astype(np.int64)).cuda()
    for d in range(s.ndim):
        shape = [1] * (1 + s.ndim)
        shape[s.ndim - d] = s.block_nx[d]
        dx = (s.xmax[d] - s.xmin[d]) / ((s.base_blocks[d] * s.block_nx[d]) * 2.0 ** (lev.double() - 1))
        i = ijk[:, d] * s.block_nx[d]
        view = [-1] + [1] * s.ndim
        loc = torch.arange(s.block_nx[d], dtype=torch.float64, device="cuda").reshape(shape)
        out.append(s.xmin[d] + ((i.view(view) + loc) + 0.5) * dx.view(view))
    return out


def _initial(f, problem: str, seed: int) -> torch.Tensor:
    """The problem's initial state with seeded parameters (the strength, position and perturbation
    that vary from run to run), conserved variables [var][leaf][z][y][x] on the GPU."""
    s, nd = f.scheme, f.scheme.ndim
    rng = np.random.default_rng([seed, 17])
    xs = _centres(f)
    shape = (f.n,) + tuple(s.block_nx[d] for d in reversed(range(nd)))
    full = lambda v: torch.full(shape, float(v), dtype=torch.float64, device="cuda")  # noqa: E731
    B = None
    if problem == "sod":
        left = (xs[0] < 0.5).expand(shape)
        rho = torch.where(left, full(rng.uniform(0.9, 1.1)), full(0.125))
        p = torch.where(left, full(rng.uniform(0.9, 1.1)), full(0.1))
        vel = [full(0.0)]
    elif problem == "kh":
        inner = (torch.abs(xs[1] - 0.5) < 0.25).expand(shape)
        g = torch.Generator(device="cuda").manual_seed(seed)
        rho, p = torch.where(inner, full(2.0), full(1.0)), full(2.5)
        noise = 2.0 * torch.rand(shape, generator=g, dtype=torch.float64, device="cuda") - 1.0
        vel = [torch.where(inner, full(0.5), full(-0.5)), 0.01 * noise]
    elif problem == "ot":
        a, tp = rng.uniform(0.9, 1.1, 4), 2.0 * math.pi
        rho, p = full(25.0 / 9.0), full(5.0 / 3.0)
        vel = [-a[0] * torch.sin(tp * xs[1]).expand(shape), a[1] * torch.sin(tp * xs[0]).expand(shape)]
        B = [-a[2] * torch.sin(tp * xs[1]).expand(shape), a[3] * torch.sin(2 * tp * xs[0]).expand(shape)]
    else:
        radius = {"dam": 2.5, "blast": 0.12 if s.max_level < 4 else 0.1, "mhdblast": 0.1}[problem]
        c = rng.uniform(-0.02, 0.02, nd) * radius
        r2 = sum((x - float(c[d])) ** 2 for d, x in enumerate(xs))
        inner = (r2 < radius * radius).expand(shape)
        vel = [full(0.0) for _ in range(nd)]
        if problem == "dam":
            rho, p = torch.where(inner, full(rng.uniform(2.0, 3.0)), full(0.5)), None
        else:
            hi = rng.uniform(50.0, 150.0) if problem == "blast" else rng.uniform(8.0, 12.0)
            rho, p = full(1.0), torch.where(inner, full(hi), full(0.1))
            if problem == "mhdblast":
                B = [full(1.0 / math.sqrt(nd)) for _ in range(nd)]
    U = torch.zeros((s.nvar,) + shape, dtype=torch.float64, device="cuda")
    U[0] = rho
    for d in range(nd):
        U[1 + d] = rho * vel[d]
    if p is not None:
        U[1 + nd] = p / (s.gamma - 1.0) + 0.5 * rho * sum(v * v for v in vel)
    if B is not None:
        U[1 + nd] += 0.5 * sum(b * b for b in B)
        for d in range(nd):
            U[2 + nd + d] = B[d]
    return U


def _fv_prepare(case, seed):
    f = _forest(case)
    g = GpuForest(f)
    if case["arith"] == "fast":
        g.set_arithmetic(N.ARITH_FAST)
    if case.get("persistent"):
        g.set_schedule(N.SCHED_PERSISTENT, 0, 0)
    if case.get("variant"):
        g.set_variant(case["variant"])
    if case.get("graph"):
        g.use_graph(True)
    if case.get("flag") == "mlp":
        g.mlp_set_weights(np.load(WEIGHTS, allow_pickle=False))
    return dict(case=case, g=g, U=_initial(f, case["problem"], seed))


def _fv_run(st):
    case, g = st["case"], st["g"]
    g.set_state(st["U"])
    if case.get("driver", "device") == "device":
        g.advance_cfl(case["steps"])
    else:
        ramp = 10 if case["problem"] == "mhdblast" else 0
        for i in range(case["steps"]):
            g.advance(g.max_dt() * courant_ramp(i, ramp))
    out = {}
    flag = case.get("flag", "none")
    if flag == "lohner":
        out["flags"], out["emax"] = g.flag_blocks(with_emax=True)
    elif flag == "mlp":
        out["flags"] = g.flag_blocks(mode=N.FLAG_MLP)
        out["logits"] = g.mlp_logits()
    if case.get("regrid"):
        h = g.regrid(out["flags"])
        out["level"] = h.forest.level
        out["U"] = h.state_tensor()
        h.close()
    else:
        out["U"] = g.state_tensor()
    return out


# floating-point operations per cell and Runge-Kutta stage: primitives, limited slopes, one flux per
# face and the update, by dimension
FLOPS = {("euler", 1): 90, ("euler", 2): 230, ("euler", 3): 400, ("mhd", 2): 420, ("mhd", 3): 900, ("poly", 2): 150}


def _fv_work(case):
    f = _forest(case)
    s = f.scheme
    cells = f.n * s.cells_per_block
    phys = {W.EULER: "euler", W.MHD: "mhd", W.POLY: "poly"}[s.physics]
    # the Courant reduction separates the steps: each reads the state once and writes it once
    return {"bytes": 16.0 * s.nvar * cells * case["steps"],
            "flops": float(FLOPS[(phys, s.ndim)] * s.rk_stages * cells * case["steps"])}


# -- the same scheme on a uniform grid in plain torch -----------------------


def _limited(lim, a, b):
    """phi(a, b), symmetric limiters: a, b the backward and forward differences."""
    same = a * b > 0
    if lim == W.MINMOD:
        v = torch.where(torch.abs(a) <= torch.abs(b), a, b)
    else:  # van Leer
        v = 2 * a * b / torch.where(same, a + b, torch.ones_like(a))
    return torch.where(same, v, torch.zeros_like(a))


class _Grid:
    """TVDLF / HLL / HLLC with limited primitive slopes and SSP-RK on a uniform grid; arrays
    [var][z][y][x], direction d on axis ndim - d."""

    def __init__(self, s):
        self.s, self.nd, self.mhd = s, s.ndim, s.physics == W.MHD
        self.dx = [(s.xmax[d] - s.xmin[d]) / (s.base_blocks[d] * s.block_nx[d]) for d in range(s.ndim)]

    def prim(self, U):
        nd, g = self.nd, self.s.gamma
        V = U.clone()
        V[1:1 + nd] = U[1:1 + nd] / U[0]
        e = U[1 + nd] - 0.5 * (U[1:1 + nd] * V[1:1 + nd]).sum(0)
        if self.mhd:
            e = e - 0.5 * (U[2 + nd:2 + 2 * nd] ** 2).sum(0)
        V[1 + nd] = (g - 1.0) * e
        return V

    def speed(self, V, d):
        nd = self.nd
        a2 = self.s.gamma * V[1 + nd] / V[0]
        if not self.mhd:
            return torch.sqrt(a2)
        b2 = (V[2 + nd:2 + 2 * nd] ** 2).sum(0) / V[0]
        bn2 = V[2 + nd + d] ** 2 / V[0]
        q = a2 + b2
        return torch.sqrt(0.5 * (q + torch.sqrt(torch.clamp(q * q - 4 * a2 * bn2, min=0.0))))

    def cons_flux(self, V, d):
        nd, g, rho, v, p = self.nd, self.s.gamma, V[0], V[1:1 + self.nd], V[1 + self.nd]
        U, F = V.clone(), torch.zeros_like(V)
        U[1:1 + nd] = rho * v
        U[1 + nd] = p / (g - 1.0) + 0.5 * rho * (v * v).sum(0)
        pt = p
        if self.mhd:
            B = V[2 + nd:2 + 2 * nd]
            U[1 + nd] = U[1 + nd] + 0.5 * (B * B).sum(0)
            pt = p + 0.5 * (B * B).sum(0)
        F[0] = rho * v[d]
        F[1:1 + nd] = U[1:1 + nd] * v[d]
        F[1 + d] = F[1 + d] + pt
        F[1 + nd] = (U[1 + nd] + pt) * v[d]
        if self.mhd:
            F[1:1 + nd] = F[1:1 + nd] - B[d] * B
            F[1 + nd] = F[1 + nd] - B[d] * (v * B).sum(0)
            F[2 + nd:2 + 2 * nd] = B * v[d] - B[d] * v
        return U, F

    def face_flux(self, L, R, d, ch):
        s, nd = self.s, self.nd
        if self.mhd:  # the GLM pair's own Riemann problem gives the normal field and psi at the face
            ib, ip = 2 + nd + d, 2 + 2 * nd
            bn = 0.5 * (L[ib] + R[ib]) - 0.5 * (R[ip] - L[ip]) / ch
            psi = 0.5 * (L[ip] + R[ip]) - 0.5 * ch * (R[ib] - L[ib])
            L, R = L.clone(), R.clone()
            L[ib], R[ib] = bn, bn
        UL, FL = self.cons_flux(L, d)
        UR, FR = self.cons_flux(R, d)
        cl, cr, ul, ur = self.speed(L, d), self.speed(R, d), L[1 + d], R[1 + d]
        if s.flux == W.TVDLF:
            F = 0.5 * ((FL + FR) - torch.maximum(torch.abs(ul) + cl, torch.abs(ur) + cr) * (UR - UL))
        else:
            SL, SR = torch.minimum(ul - cl, ur - cr), torch.maximum(ul + cl, ur + cr)
            if s.flux == W.HLL:
                mid = (SR * FL - SL * FR + SL * SR * (UR - UL)) / (SR - SL)
                F = torch.where(SL >= 0, FL, torch.where(SR > 0, mid, FR))
            else:
                pl, pr, ml, mr = L[1 + nd], R[1 + nd], L[0] * (SL - ul), R[0] * (SR - ur)
                SM = ((pr - pl) + ul * ml - ur * mr) / (ml - mr)

                def star(V, U, S, u, p, m):
                    Us = U * 0
                    Us[0] = m / (S - SM)
                    Us[1:1 + nd] = Us[0] * V[1:1 + nd]
                    Us[1 + d] = Us[0] * SM
                    Us[1 + nd] = ((S - u) * U[1 + nd] - p * u + (p + m * (SM - u)) * SM) / (S - SM)
                    return Us

                FsL = FL + SL * (star(L, UL, SL, ul, pl, ml) - UL)
                FsR = FR + SR * (star(R, UR, SR, ur, pr, mr) - UR)
                F = torch.where(SL >= 0, FL, torch.where(SM >= 0, FsL, torch.where(SR > 0, FsR, FR)))
        if self.mhd:
            F[ib], F[ip] = psi, ch * ch * bn
        return F

    def pad(self, V, ax):
        """Two ghost layers along one axis."""
        n = V.shape[ax]
        if self.s.bc == W.PERIODIC:
            return torch.cat([V.narrow(ax, n - 2, 2), V, V.narrow(ax, 0, 2)], ax)
        lo, hi = V.narrow(ax, 0, 1), V.narrow(ax, n - 1, 1)
        return torch.cat([lo, lo, V, hi, hi], ax)

    def rhs(self, U, ch):
        V, acc = self.prim(U), 0
        for d in range(self.nd):
            ax, n = self.nd - d, U.shape[self.nd - d]
            P = self.pad(V, ax)
            dif = P.narrow(ax, 1, n + 3) - P.narrow(ax, 0, n + 3)
            slope = _limited(self.s.limiter, dif.narrow(ax, 0, n + 2), dif.narrow(ax, 1, n + 2))
            up, low = P.narrow(ax, 1, n + 2) + 0.5 * slope, P.narrow(ax, 1, n + 2) - 0.5 * slope
            F = self.face_flux(up.narrow(ax, 0, n + 1), low.narrow(ax, 1, n + 1), d, ch)
            acc = acc + (F.narrow(ax, 1, n) - F.narrow(ax, 0, n)) / self.dx[d]
        return acc

    def advance(self, U, steps):
        s = self.s
        for _ in range(steps):
            V = self.prim(U)
            sp = [torch.abs(V[1 + d]) + self.speed(V, d) for d in range(self.nd)]
            dt = s.cfl / float(sum(c / self.dx[d] for d, c in enumerate(sp)).max())
            ch = max(float(c.max()) for c in sp)
            U1 = U - dt * self.rhs(U, ch)
            if s.rk_stages == 2:
                U = 0.5 * U + 0.5 * (U1 - dt * self.rhs(U1, ch))
            else:
                U2 = 0.75 * U + 0.25 * (U1 - dt * self.rhs(U1, ch))
                U = (1.0 / 3.0) * U + (2.0 / 3.0) * (U2 - dt * self.rhs(U2, ch))
            if self.mhd:
                U[-1] = U[-1] * math.exp(-dt * ch / s.glm_cr)
        return U


def _fv_exact(case, seed):
    if case["problem"] not in ("sod", "kh", "ot"):
        return None  # refined forests
    f = _forest(case)
    s, nd = f.scheme, f.scheme.ndim
    U = _initial(f, case["problem"], seed)
    grid = torch.zeros([s.nvar] + [s.base_blocks[d] * s.block_nx[d] for d in reversed(range(nd))],
                       dtype=torch.float64, device=U.device)
    place = [tuple([slice(None)] + [slice(int(c[d]) * s.block_nx[d], (int(c[d]) + 1) * s.block_nx[d])
                                    for d in reversed(range(nd))]) for c in f.ijk]
    for b, at in enumerate(place):
        grid[at] = U[:, b]
    grid = _Grid(s).advance(grid, case["steps"])
    return {"U": torch.stack([grid[at] for at in place], dim=1)}


# ---------------------------------------------------------------------------
# reaction-diffusion and elliptic cases
# ---------------------------------------------------------------------------

SCHEMES = {"euler": M.EULER, "midpoint": M.MIDPOINT, "split": M.SPLIT, "imex": M.IMEX}
PARAMS = {"schnakenberg": dict(model=M.SCHNAKENBERG, Du=0.05, Dv=1.0, p1=100.0, p2=0.1305, p3=0.7695),
          "gray_scott": dict(model=M.GRAY_SCOTT, Du=2e-5, Dv=1e-5, p1=0.046, p2=0.063, p3=0.0)}


def _rd_fields(model, xs, seed):
    rng = np.random.default_rng([seed, 29])
    if model == "schnakenberg":
        a, b = 0.1305, 0.7695
        c, amp = rng.uniform(0.3, 0.6, len(xs)), rng.uniform(0.8, 1.2)
        u = a + b + amp * torch.exp(-100.0 * sum((x - float(c[d])) ** 2 for d, x in enumerate(xs)))
        return u, torch.full_like(u, b / (a + b) ** 2)
    g = 0
    for c in ((0.5, 0.5, 0.5), (0.55, 0.6, 0.5)):
        c = np.asarray(c) + rng.uniform(-0.03, 0.03, 3)
        g = g + 0.5 * torch.exp(-25.0 * sum((x - float(c[d])) ** 2 for d, x in enumerate(xs)))
    return 1.0 - g, g.clone()


def _rd_setup(case):
    """(dt, domain length, boundary): Schnakenberg has zero-flux walls, Gray-Scott is periodic;
    explicit steps stay below their diffusive limit."""
    model = case["model"]
    length, bc = (1.0, M.NEUMANN) if model == "schnakenberg" else (2.0, M.PERIODIC)
    dt = case["dt"]
    if case["scheme"] in ("euler", "midpoint"):
        p = PARAMS[model]
        dt = min(dt, 0.4 * (length / case["n"]) ** 2 / (2 * case["ndim"] * max(p["Du"], p["Dv"])))
    return dt, length, bc


def _rd_initial(case, seed):
    n, nd = case["n"], case["ndim"]
    _, length, _ = _rd_setup(case)
    c = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) * (length / n)
    xs = [c.view([-1 if a == nd - 1 - d else 1 for a in range(nd)]).expand((n,) * nd) for d in range(nd)]
    u, v = _rd_fields(case["model"], xs, seed)
    return u.contiguous(), v.contiguous()


def _rd_prepare(case, seed):
    u, v = _rd_initial(case, seed)
    dt, length, bc = _rd_setup(case)
    mg = M.GpuMultigrid(case["ndim"], case["n"], bc, length, nfields=2)
    return dict(case=case, s=mg, u0=u, v0=v, u=u.clone(), v=v.clone(), dt=dt, p=PARAMS[case["model"]])


def _rdf_prepare(case, seed):
    f = _gs_forest(case["base"], case["levels"])
    u, v = _rd_fields("gray_scott", [x.contiguous() for x in torch.broadcast_tensors(*_centres(f))], seed)
    dt = case["dt"] if case["scheme"] in ("imex", "split") else min(case["dt"], 0.05)
    return dict(case=case, s=M.GpuForestMultigrid(f, 2.0, M.PERIODIC), u0=u, v0=v, u=u.clone(), v=v.clone(), dt=dt,
                p=PARAMS["gray_scott"])


@functools.lru_cache(maxsize=None)
def _gs_forest(base, levels):
    return W.gray_scott_amr(base, levels)[0]


def _rd_run(st):
    case = st["case"]
    st["u"].copy_(st["u0"])
    st["v"].copy_(st["v0"])
    tol = 1e-7  # the paper's stopping rule
    st["s"].rd_step(st["u"], st["v"], st["dt"], SCHEMES[case["scheme"]], st["p"], nsteps=case["steps"], tol=tol)
    return st["u"], st["v"]


def _rd_exact(case, seed):
    n, nd = case["n"], case["ndim"]
    u, v = _rd_initial(case, seed)
    dt, length, bc = _rd_setup(case)
    k = torch.arange(n, dtype=torch.float64, device=u.device)
    h2 = (n / length) ** 2
    i = k[:, None] + 0.5
    if bc == M.NEUMANN:  # cosine modes of the cell-centred grid
        Q = torch.cos(math.pi * i * k / n) * math.sqrt(2.0 / n)
        Q[:, 0] = math.sqrt(1.0 / n)
        lam1 = -4.0 * h2 * torch.sin(math.pi * k / (2 * n)) ** 2
    else:  # real Fourier modes
        w = torch.minimum(k, n - k)
        Q = torch.where(k <= n // 2, torch.cos(2 * math.pi * i * w / n), torch.sin(2 * math.pi * i * w / n))
        Q[:, n // 2] = torch.sin(math.pi * i[:, 0])
        Q = Q / torch.linalg.norm(Q, dim=0)
        lam1 = -4.0 * h2 * torch.sin(math.pi * w / n) ** 2
    eig = sum(lam1.view([-1 if a == d else 1 for a in range(nd)]) for d in range(nd))

    def modes(x, A):
        for a in range(nd):
            x = torch.movedim(torch.tensordot(A, x, dims=([0], [a])), 0, a)
        return x

    def lap(x):
        out = 0
        for a in range(nd):
            lo, hi = torch.roll(x, 1, a), torch.roll(x, -1, a)
            if bc == M.NEUMANN:
                lo.narrow(a, 0, 1).copy_(x.narrow(a, 0, 1))
                hi.narrow(a, n - 1, 1).copy_(x.narrow(a, n - 1, 1))
            out = out + ((lo + hi) - 2.0 * x) * h2
        return out

    p = PARAMS[case["model"]]

    def react(u, v):
        if case["model"] == "schnakenberg":
            return p["p1"] * (p["p2"] - u + u * u * v), p["p1"] * (p["p3"] - u * u * v)
        return -u * v * v + p["p1"] * (1.0 - u), u * v * v - (p["p1"] + p["p2"]) * v

    D = (p["Du"], p["Dv"])

    def full(w):
        return [r + D[c] * lap(w[c]) for c, r in enumerate(react(*w))]

    def implicit(w, tau):  # (1 - tau D lap) x = w
        return [modes(modes(x, Q) / (1.0 - tau * D[c] * eig), Q.t().contiguous()) for c, x in enumerate(w)]

    w = [u, v]
    for _ in range(case["steps"]):
        if case["scheme"] == "midpoint":
            k1 = full(w)
            k2 = full([x + 0.5 * dt * d for x, d in zip(w, k1)])
            w = [x + dt * d for x, d in zip(w, k2)]
        elif case["scheme"] == "split":
            w = implicit([x + dt * r for x, r in zip(w, react(*w))], dt)
        else:
            r, F = react(*w), full(w)
            s = implicit([x + dt * r[c] + 0.5 * dt * D[c] * lap(x) for c, x in enumerate(w)], 0.5 * dt)
            w = [x + 0.5 * dt * (a + b) for x, a, b in zip(w, F, full(s))]
    return w[0], w[1]


@functools.lru_cache(maxsize=None)
def _helm_forest(ndim, base, levels, radius, bc):
    s = W.fmg_scheme(base=base, max_level=levels, bc=bc, ndim=ndim)
    return W.fmg_forest(s, centre=(0.45, 0.52, 0.48), radius=radius)


def _helm_of(case):
    return _helm_forest(case["ndim"], case["base"], case["levels"], case["radius"],
                        M.PERIODIC if case["bc"] == "periodic" else M.NEUMANN)


def _helm_prepare(case, seed):
    f = _helm_of(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng([seed, 41])
    xs = _centres(f)
    c = rng.uniform(0.3, 0.7, case["ndim"])
    rhs = torch.exp(-40.0 * sum((x - float(c[d])) ** 2 for d, x in enumerate(xs)))
    rhs = (rhs + rng.uniform(0.5, 1.0) * torch.cos(2 * math.pi * xs[0]) * torch.cos(4 * math.pi * xs[1])).contiguous()
    rhs += 0.1 * (2.0 * torch.rand(rhs.shape, generator=g, dtype=torch.float64, device="cuda") - 1.0)
    solver = M.GpuForestMultigrid(f, 1.0, M.PERIODIC if case["bc"] == "periodic" else M.NEUMANN)
    return dict(case=case, s=solver, f=rhs, phi=torch.zeros_like(rhs))


def _helm_run(st):
    st["phi"].zero_()
    st["s"].solve(st["f"], st["phi"], st["case"]["lam"])
    return st["phi"]


# ---------------------------------------------------------------------------
# training of the refinement flagger
# ---------------------------------------------------------------------------

ADAM_T0 = 1000  # steps already taken: an epoch in the middle of a training


def _train_data(case, seed):
    X, y = W.mlp_random_features(seed, case["samples"])
    # labels that the features carry, as the estimator's classes do
    x0 = (X[:, 0].astype(np.uint32) << 16).view(np.float32)
    y = np.where(x0 > 0.4, 1.0, np.where(x0 < -0.2, -1.0, y * (np.abs(x0) > 0.3))).astype(np.float32)
    rng = np.random.default_rng([seed, 53])
    w = W.mlp_init(seed)
    m = (1e-3 * rng.standard_normal(w.size)).astype(np.float32)
    v = (1e-5 * rng.uniform(0.5, 2.0, w.size)).astype(np.float32)
    return X, y, w, m, v


def _train_prepare(case, seed):
    X, y, w, m, v = _train_data(case, seed)
    tr = L.Trainer(X, y, batch=case["batch"], seed=seed % 1000)
    return dict(case=case, tr=tr, start=[torch.from_numpy(a).to(tr.dev) for a in (w, m, v)])


def _train_run(st):
    tr = st["tr"]
    for to, a in zip((tr.w, tr.m, tr.v), st["start"]):
        to.copy_(a)
    tr.t = ADAM_T0
    loss = tr.epoch(0)
    return {"w": tr.w, "m": tr.m, "v": tr.v, "loss": loss, "losses": tr.loss}


def _train_exact(case, seed):
    X, y, w, m, v = _train_data(case, seed)
    n, B = case["samples"], case["batch"]
    order = np.random.default_rng((seed % 1000) * 1000).permutation(n)
    npos, nneg = float(np.sum(y > 0.5)), float(np.sum(y < -0.5))
    pw = (max(1.0, (n - npos) / max(npos, 1.0)), max(0.05, (n - nneg) / max(nneg, 1.0)))
    t64 = lambda a: torch.from_numpy(np.asarray(a)).to("cuda").double()  # noqa: E731
    x = t64((X.astype(np.uint32) << 16).view(np.float32))
    lab = t64(y)
    w, m, v = t64(w), t64(m), t64(v)
    nin, nh, no = W.MLP_NIN, W.MLP_NH, W.MLP_NOUT
    sizes = [nh * nin, nh, nh * nh, nh, no * nh, no]
    losses = []
    for b in range((n + B - 1) // B):
        idx = torch.from_numpy(order[b * B:(b + 1) * B]).to("cuda")
        xb, yb = x[idx], torch.stack([lab[idx] > 0.5, lab[idx] < -0.5], 1).double()
        W1, b1, W2, b2, W3, b3 = torch.split(w, sizes)
        W1, W2, W3 = W1.view(nh, nin), W2.view(nh, nh), W3.view(no, nh)
        h1 = torch.relu(xb @ W1.t() + b1)
        h2 = torch.relu(h1 @ W2.t() + b2)
        z = h2 @ W3.t() + b3
        pwt = torch.tensor(pw, dtype=torch.float64, device="cuda")
        sp = torch.nn.functional.softplus
        losses.append(((pwt * yb * sp(-z) + (1 - yb) * sp(z)).sum() / len(idx)))
        sg = torch.sigmoid(z)
        dz = ((1 - yb) * sg - pwt * yb * (1 - sg)) / len(idx)
        d2 = (dz @ W3) * (h2 > 0)
        d1 = (d2 @ W2) * (h1 > 0)
        gr = torch.cat([(d1.t() @ xb).flatten(), d1.sum(0), (d2.t() @ h1).flatten(), d2.sum(0),
                        (dz.t() @ h2).flatten(), dz.sum(0)])
        t = ADAM_T0 + b + 1
        m = 0.9 * m + 0.1 * gr
        v = 0.999 * v + 0.001 * gr * gr
        w = w - 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    losses = torch.stack(losses)
    return {"w": w, "m": m, "v": v, "loss": float(losses.mean()), "losses": losses}


# ---------------------------------------------------------------------------
# the entry points of this file
# ---------------------------------------------------------------------------

def prepare(case: dict, seed: int):
    return {"fv": _fv_prepare, "rd": _rd_prepare, "rdf": _rdf_prepare, "helm": _helm_prepare,
            "train": _train_prepare}[case["kind"]](case, seed)


def run(state):
    return {"fv": _fv_run, "rd": _rd_run, "rdf": _rd_run, "helm": _helm_run,
            "train": _train_run}[state["case"]["kind"]](state)


def work(case: dict) -> dict:
    kind = case["kind"]
    if kind == "fv":
        return _fv_work(case)
    if kind == "train":
        # forward and both backward products of the three layers, on each sample once
        return {"bytes": case["samples"] * 260.0, "flops": case["samples"] * 6.0 * (128 * 64 + 64 * 64 + 64 * 2)}
    if kind == "rd":
        cells = case["n"] ** case["ndim"]
    elif kind == "rdf":
        cells = 256 * _gs_forest(case["base"], case["levels"]).n
    else:
        f = _helm_of(case)
        cells = f.n * 16 ** case["ndim"]
        # right-hand side in, solution out; a red-black sweep, its residual and correction per cycle at least
        return {"bytes": 16.0 * cells, "flops": 40.0 * cells}
    # both species read and written once a step; reaction, diffusion and one sweep of each solve at least
    return {"bytes": 32.0 * cells * case["steps"], "flops": 80.0 * cells * case["steps"]}


def exact(case: dict, seed: int):
    kind = case["kind"]
    if kind == "fv":
        return _fv_exact(case, seed)
    if kind == "rd":
        return _rd_exact(case, seed)
    if kind == "train":
        return _train_exact(case, seed)
    return None  # the composite operator of a refined forest
