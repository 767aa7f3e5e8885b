"""The work whose speed is measured: what a program does with this library through its public
Python entry points (paper_1608_06721_amd.nmg and .adjoint), from the smallest calls to the
benchmark solve.

A case is a dict of plain values; "kind" names the call:

  residual  one residual and its l1 norm, without a context (a monitor or a time loop's check)
  blu       one nonlinear smoothing sweep of a state
  step      one Newton linearization (residual, Jacobian, coarse levels) and its multigrid
            cycles, for programs that drive their own Newton loop
  solve     a whole steady solve from given data (channel, dry hill or a 1D flow)
  batch     independent steady solves of uneven size in one call (ensembles)
  adjoint   an adjoint solve and the bed gradient at a given steady state
  gradient  a steady state and the bed gradient of a gauge misfit by automatic differentiation

Grids are those of this repository's workloads (channel, dry hill, 1D bump and smooth flow) and
others of the same kind; beds, states and discharges come from the seed.
"""
import math

import numpy as np
import torch

from paper_1608_06721_amd import adjoint, nmg
from paper_1608_06721_amd import workloads as W

TOL = 1e-10


def _case(name, kind, nx, ny, levels, **kw):
    c = dict(name=name, kind=kind, nx=nx, ny=ny, levels=levels, gamma=1, fp32=False, flux="llf")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a monitor's residual of a small grid (latency of two launches)
        _case("residual_small", "residual", 64, 48, 0),
        # the 1D example at its usual size: a whole solve of launches that are nearly empty
        _case("solve_1d", "solve", 200, 1, 3, setting="bump", flux="hll"),
        # a nonlinear smoothing sweep on an ordinary grid
        _case("blu_512", "blu", 512, 384, 0),
        # a linearization and its cycles on a small grid with odd coarse levels
        _case("step_small", "step", 96, 80, 3),
        # the default cycle on an ordinary grid, single-precision hierarchy
        _case("step_fp32", "step", 512, 256, 3, fp32=True),
        # a ragged grid (125 x 75 at the bottom) with the HLL flux
        _case("step_ragged", "step", 1000, 600, 3, flux="hll"),
        # the largest linearization: W-cycles on the benchmark's mesh
        _case("step_large", "step", 1024, 1024, 5, gamma=2),
        # the wet/dry example with its nested initial guess
        _case("solve_hill", "solve", 256, 128, 4, setting="hill", gamma=2),
        # the benchmark solve: two emergent islands, nested initial guess, W-cycles
        _case("solve_islands", "solve", 1024, 1024, 5, setting="islands", gamma=2),
        # an ensemble of uneven channels, single-precision hierarchy
        _case("batch_fp32", "batch", 384, 384, 4, count=24, gamma=2, fp32=True),
        # the backward half of a gradient: adjoint and bed product on an ordinary grid
        _case("adjoint_512", "adjoint", 512, 512, 5, gamma=2),
        # both directions of a gradient on a small grid
        _case("gradient_128", "gradient", 128, 64, 3, gamma=2),
    ]


def _size(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over its logarithm."""
    n = round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)
    return max(1, n) * step


def draw(rng):
    kind = rng.choice(["residual", "blu", "step", "step", "solve", "solve", "batch", "adjoint",
                       "gradient"])
    flux = rng.choice(["llf", "llf", "hll", "hllc"])
    gamma = rng.choice([1, 2])
    fp32 = rng.random() < 0.4
    if kind in ("residual", "blu"):
        c = _case("", kind, _size(rng, 24, 1024, 1), _size(rng, 24, 1024, 1), 0, flux=flux)
    elif kind == "step":
        nl = rng.choice([2, 3, 4, 5])
        c = _case("", kind, _size(rng, 32, 1024, 1 << nl), _size(rng, 32, 1024, 1 << nl), nl,
                  gamma=gamma, fp32=fp32, flux=flux)
    elif kind == "solve":
        setting = rng.choice(["bump", "smooth", "hill", "channel"])
        nl = rng.choice([3, 4])
        if setting in ("bump", "smooth"):
            c = _case("", kind, _size(rng, 64, 1024, 8), 1, 3, setting=setting,
                      flux=rng.choice(["llf", "hll"]))
        else:
            nx = _size(rng, 64, 320, 1 << nl)
            c = _case("", kind, nx, max(1, nx // (2 << nl)) << nl, nl, setting=setting,
                      gamma=2, fp32=fp32)
    elif kind == "batch":
        c = _case("", kind, _size(rng, 64, 256, 16), _size(rng, 64, 256, 16), 4,
                  count=rng.randint(2, 16), gamma=2, fp32=fp32)
    else:
        nl = rng.choice([2, 3])
        c = _case("", kind, _size(rng, 24, 256, 1 << nl), _size(rng, 24, 256, 1 << nl), nl, gamma=2)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs

def _params(case, dim, **kw):
    flux = {"hll": W.HLL, "llf": W.LLF, "hllc": W.HLLC}[case["flux"]]
    return W.default_params(dim, flux=flux, n_levels=case["levels"], gamma=case["gamma"],
                            inner_fp32=int(case["fp32"]), **kw)


def _bed(nx, ny, rng, amp=0.3, mounds=2, mound_amp=1.1, mound_width=0.5):
    """A channel bed on [0, 10] x [0, 2] of the kind that workloads.channel_bed draws: seeded
    Gaussians and emergent mounds."""
    x = W.cell_centres(0.0, 10.0, nx)[None, :]
    y = W.cell_centres(0.0, 2.0, ny)[:, None]

    def gauss(a, w, cx, cy):    # separable: one exponential per column and row
        return a * (np.exp(-((y - cy) / w) ** 2) * np.exp(-((x - cx) / w) ** 2))

    z = np.zeros((ny, nx))
    for _ in range(16):
        z += gauss(rng.uniform(0.0, amp), rng.uniform(0.2, 0.6), rng.uniform(0, 10),
                   rng.uniform(0, 2))
    z *= min(1.0, 1.5 * amp / z.max())
    for k in range(mounds):
        z += gauss(mound_amp, mound_width, 3.5 + 2.5 * k + rng.uniform(-0.5, 0.5),
                   rng.uniform(0.5, 1.5))
    return z


def _channel(case, nx, ny, z, q=1.0, **kw):
    U0 = np.zeros((3, ny, nx))
    U0[0] = np.maximum(0.0, 1.0 - z)
    bc = [W.open_q(q, 0.0), W.open_h(1.0), W.wall(), W.wall()]
    return W.Problem("channel", 2, nx, ny, 0.0, 10.0, 0.0, 2.0, bc, _params(case, 2, **kw), z, U0)


def _flow(prob, rng):
    """A moving state over the bed of `prob`: the water surface and the velocities vary smoothly."""
    x = np.linspace(0.0, 1.0, prob.nx)[None, :]
    y = np.linspace(0.0, 1.0, prob.ny)[:, None]
    a, b, c = rng.uniform(0.0, 2.0 * math.pi, 3)
    eta = 1.0 + 0.02 * np.sin(7 * x + a) * np.cos(3 * y + b)
    U = np.zeros_like(prob.U0)
    U[0] = np.maximum(0.0, eta - prob.z)
    U[1] = U[0] * (0.8 + 0.2 * np.sin(5 * x + 2 * y + c))
    U[2] = U[0] * 0.1 * np.cos(4 * x + 6 * y + a)
    return U


def _problem(case, seed):
    """The problem of one case and seed (grid, boundary data, bed, initial data)."""
    rng = np.random.default_rng(seed)
    nx, ny, kind = case["nx"], case["ny"], case["kind"]
    if kind == "solve":
        setting = case["setting"]
        if setting in ("bump", "smooth"):
            p = (W.bump_1d if setting == "bump" else W.smooth_1d)(nx)
            p.params = _params(case, 1, max_newton=100)
            p.z = p.z * rng.uniform(0.9, 1.0)
            p.U0[0, 0] = (2.0 if setting == "bump" else 1.0) - p.z[0]
            return p
        if setting == "hill":
            p = W.dry_hill(nx, ny)
            p.params = _params(case, 2, eps_p=0.2, max_newton=40)
            p.bc[0] = W.open_q(rng.uniform(0.095, 0.105), 0.0)
            return p
        if setting == "islands":
            p = W.benchmark_channel(nx, n_levels=case["levels"], gamma=case["gamma"],
                                    max_newton=100)
            p.bc[0] = W.open_q(rng.uniform(0.999, 1.001), 0.0)
            return p
        return _channel(case, nx, ny, _bed(nx, ny, rng, amp=0.2, mound_amp=0.3),
                        rng.uniform(0.5, 1.0), max_newton=60)
    if kind in ("adjoint", "gradient"):     # submerged beds: every seed has a steady state
        return _channel(case, nx, ny, _bed(nx, ny, rng, amp=0.03, mound_amp=0.05,
                                                mound_width=0.8),
                        rng.uniform(0.4, 0.6), max_newton=400)
    p = _channel(case, nx, ny, _bed(nx, ny, rng))
    p.U0 = _flow(p, rng)
    return p


def _batch(case, seed):
    rng, sizes = np.random.default_rng(seed), np.random.default_rng(case["count"])
    step = 1 << case["levels"]
    probs = []
    for _ in range(case["count"]):          # the grids are the case's, the data the seed's
        nx = max(2, int(case["nx"] * sizes.uniform(0.3, 1.0)) // step) * step
        ny = max(2, int(case["ny"] * sizes.uniform(0.3, 1.0)) // step) * step
        z = _bed(nx, ny, rng, amp=0.2, mound_amp=0.4)
        probs.append(_channel(case, nx, ny, z, rng.uniform(0.5, 1.0), max_newton=60))
    return probs


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "batch":
        probs = _batch(case, seed)
        s.update(batch=nmg.Batch(probs), z=[_dev(p.z) for p in probs],
                 U0=[_dev(p.U0) for p in probs])
        s["U"] = [torch.empty_like(u) for u in s["U0"]]
        return s
    p = _problem(case, seed)
    s.update(prob=p, z=_dev(p.z), U0=_dev(p.U0))
    s["U"] = torch.empty_like(s["U0"])
    if kind == "residual":
        s.update(R=torch.empty_like(s["U0"]),
                 norm=torch.empty(1, dtype=torch.float64, device="cuda"))
        return s
    s["ctx"] = nmg.Context.from_problem(p)
    if kind == "step":
        s.update(R=torch.empty_like(s["U0"]), dU=torch.empty_like(s["U0"]))
    elif kind == "adjoint":
        s["U"].copy_(s["U0"])
        s["ctx"].newton_mg_solve(s["z"], s["U"], TOL)
        rng = np.random.default_rng(seed + 1)
        s["g"] = _dev(rng.standard_normal(p.U0.shape) * (p.U0[0] > 0.05))
    elif kind == "gradient":
        rng = np.random.default_rng(seed + 1)
        s["gauges"] = _dev(np.sort(rng.choice(p.nx * p.ny, 32, replace=False)))
        s["target"] = _dev(rng.uniform(0.95, 1.05, 32))
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "residual":
        nmg.residual_noalloc(s["prob"], s["z"], s["U0"], s["R"], s["norm"])
        return {"R": s["R"], "norm": s["norm"]}
    if kind == "blu":
        s["U"].copy_(s["U0"])
        s["ctx"].blu_sweep(s["z"], s["U"])
        return {"U": s["U"]}
    if kind == "step":
        norm = s["ctx"].assemble_residual_jacobian(s["z"], s["U0"], s["R"])
        s["dU"].zero_()
        s["ctx"].mg_vcycle(s["dU"], 3)
        return {"R": s["R"], "norm": norm, "dU": s["dU"]}
    if kind == "solve":
        s["U"].copy_(s["U0"])
        st = s["ctx"].newton_mg_solve(s["z"], s["U"], TOL)
        return {"U": s["U"], "steps": st["newton_steps"], "sweeps": st["init_sweeps"],
                "pinned": st["n_pinned"], "ok": st["status"] == "OK"}
    if kind == "batch":
        for u, u0 in zip(s["U"], s["U0"]):
            u.copy_(u0)
        st = s["batch"].newton_mg_solve(s["z"], s["U"], TOL)
        return {"U": s["U"], "steps": np.array([r["newton_steps"] for r in st]),
                "ok": np.array([r["status"] == "OK" for r in st])}
    if kind == "adjoint":
        lam, cycles, _ = s["ctx"].adjoint_solve(s["z"], s["U"], s["g"], tol=1e-12,
                                                max_cycles=200, krylov=30)
        return {"lam": lam, "dz": s["ctx"].bed_vjp(s["z"], s["U"], lam), "cycles": cycles}
    z = s["z"].clone().requires_grad_(True)
    U = adjoint.steady_state(s["ctx"], z, s["U0"], TOL)
    loss = adjoint.gauge_misfit(U, z, s["gauges"], s["target"])
    loss.backward()
    return {"U": U.detach(), "loss": loss.detach(), "dz": z.grad}


# ---------------------------------------------------------------------------
# What a pass cannot do without

def work(case):
    kind, n = case["kind"], case["nx"] * case["ny"]
    dim = 1 if case["ny"] == 1 else 2
    nc = dim + 1
    flux = 40.0                                     # operations of one face's edge term
    faces, entries = 2 * dim, (2 * dim + 1) * nc * nc
    assembly = faces * (1 + 2 * nc) * flux + 3 * entries
    sweep = 2.0 * entries                           # one symmetric iteration's cell, per colour
    cycle = (2 + 2) * 2 * sweep * (1.34 if case["gamma"] == 1 else 2.0)
    blu = 2 * faces * (1 + nc) * flux
    newton = blu + assembly + 3 * cycle
    if kind == "residual":
        return {"bytes": 8.0 * n * (1 + 2 * nc), "flops": n * faces * flux}
    if kind == "blu":
        return {"bytes": 8.0 * n * (1 + 2 * nc), "flops": n * blu}
    if kind == "step":
        return {"bytes": 8.0 * n * (1 + 3 * nc), "flops": n * (assembly + 3 * cycle)}
    if kind == "solve":         # of the order of ten Newton steps
        return {"bytes": 8.0 * n * (1 + 2 * nc), "flops": n * 10 * newton}
    if kind == "batch":         # instances of 0.65 of either side on average
        m = 0.42 * n * case["count"]
        return {"bytes": 8.0 * m * (1 + 2 * nc), "flops": m * 10 * newton}
    adj = assembly + 15 * cycle + faces * 4 * flux
    if kind == "adjoint":
        return {"bytes": 8.0 * n * (2 + 3 * nc), "flops": n * adj}
    return {"bytes": 8.0 * n * (2 + 2 * nc), "flops": n * (10 * newton + adj)}


# ---------------------------------------------------------------------------
# The same results in plain torch, FP64: whole arrays at a time, the method written out from its
# definition (hydrostatic reconstruction, face fluxes, forward differences, red-black block
# Gauss-Seidel, Galerkin multigrid).

class _Plain:
    def __init__(self, p):
        self.p, self.q = p, p.params
        self.nc, self.nf = (2, 2) if p.dim == 1 else (3, 4)
        dx, dy = (p.x1 - p.x0) / p.nx, (p.y1 - p.y0) / p.ny
        self.e = [1.0] * 2 if p.dim == 1 else [dy, dy, dx, dx]
        self.z = _dev(p.z)

    @staticmethod
    def colour(ny, nx, c):
        j, i = torch.meshgrid(torch.arange(ny, device="cuda"), torch.arange(nx, device="cuda"),
                              indexing="ij")
        return (i + j) % 2 == c

    def side(self, U, z):
        h = U[0]
        wet = h > self.q["h_eps"]
        u = torch.where(wet, U[1] / h, 0.0)
        v = torch.where(wet, U[2] / h, 0.0) if self.nc == 3 else torch.zeros_like(u)
        return h, u, v, z

    def ghost(self, f, s):
        (kind, hb, qb, tb), g = self.p.bc[f], self.q["g"]
        h, u, v, z = s
        sgn = -1.0 if f in (0, 2) else 1.0
        un, ut = (sgn * u, v) if f < 2 else (sgn * v, u)
        if kind == W.REFLECT:
            hg, ug, tg = h, -un, ut
        elif kind == W.SLIP:
            hg, ug, tg = h, torch.zeros_like(un), ut
        else:
            sup = (h > self.q["h_eps"]) & (u * u + v * v >= g * h)
            K = un + 2.0 * torch.sqrt(g * h)
            if not math.isnan(qb):
                c = torch.clamp(K, min=0.0) + max(1.0, g * qb)
                for _ in range(100):
                    c = torch.minimum(c, c - ((2 * c - K) * c * c - g * qb) / ((6 * c - 2 * K) * c))
                hg = c * c / g
                ug, tg = -qb / hg, torch.full_like(h, 0.0 if math.isnan(tb) else tb)
            else:
                hg = torch.full_like(h, hb)
                ug, tg = K - 2.0 * math.sqrt(g * hb), ut
            out = sup & (un >= 0)
            hg, ug, tg = torch.where(out, h, hg), torch.where(out, un, ug), torch.where(out, ut, tg)
        return (hg, sgn * ug, tg, z) if f < 2 else (hg, tg, sgn * ug, z)

    @staticmethod
    def shift(a, f, fill=None):
        """Values of the neighbour across face f; `fill` (or the cell itself) at the boundary."""
        d = -1 if f < 2 else -2
        out = torch.roll(a, 1 if f in (0, 2) else -1, d)
        k = 0 if f in (0, 2) else a.shape[d] - 1
        out.select(d, k).copy_(a.select(d, k) if fill is None else torch.full_like(a.select(d, k), fill))
        return out

    def other(self, f, own, s):
        """The state across face f: the neighbour's s, the ghost of `own` at the boundary."""
        out = [self.shift(a, f) for a in s]
        d, k = (-1 if f < 2 else -2), (0 if f in (0, 2) else -1)
        for a, b in zip(out, self.ghost(f, tuple(x.select(d, k) for x in own))):
            a.select(d, k).copy_(b)
        return out

    def flux(self, ax, L, R):
        q, g = self.q, self.q["g"]
        F, Q, c, un = [], [], [], []
        for h, u, v in (L, R):
            n = (u, v)[ax]
            m, pr = h * n, 0.5 * g * h * h
            F.append([m, m * u + (pr if ax == 0 else 0), m * v + (pr if ax == 1 else 0)])
            Q.append([h, h * u, h * v])
            c.append(torch.sqrt(g * h))
            un.append(n)
        if q["flux"] == W.LLF:
            s = torch.maximum(un[0].abs() + c[0], un[1].abs() + c[1])
            s = s + q["eps_r"] * torch.maximum(c[0], c[1])
            return [0.5 * ((F[0][k] + F[1][k]) - s * (Q[1][k] - Q[0][k])) for k in range(3)]
        us = (un[0] + un[1]) * 0.5 + c[0] - c[1]
        cs = torch.abs((c[0] + c[1]) + (un[0] - un[1]) * 0.5) * 0.5
        sL = torch.where(L[0] == 0, un[1] - 2 * c[1], torch.minimum(un[0] - c[0], us - cs))
        sR = torch.where(R[0] == 0, un[0] + 2 * c[0], torch.maximum(un[1] + c[1], us + cs))
        out = [((sR * F[0][k] - sL * F[1][k]) + sL * sR * (Q[1][k] - Q[0][k])) / (sR - sL)
               for k in range(3)]
        if q["flux"] == W.HLLC:
            num = sL * R[0] * (un[1] - sR) - sR * L[0] * (un[0] - sL)
            den = R[0] * (un[1] - sR) - L[0] * (un[0] - sL)
            left = torch.where(den != 0, num / den, 0.0) >= 0
            out[2 - ax] = torch.where(left, L[2 - ax], R[2 - ax]) * out[0]
        return [torch.where(sL >= 0, F[0][k], torch.where(sR <= 0, F[1][k], out[k]))
                for k in range(3)]

    def term(self, f, own, oth):
        """Edge term of face f for the cell on side `own`, and whether both depths there are 0."""
        ax, left = f // 2, f in (1, 3)
        L, R = (own, oth) if left else (oth, own)
        zM = torch.maximum(L[3], R[3])
        hL, hR = torch.clamp(L[0] + L[3] - zM, min=0.0), torch.clamp(R[0] + R[3] - zM, min=0.0)
        T = self.flux(ax, (hL, L[1], L[2]), (hR, R[1], R[2]))
        ho = hL if left else hR
        T[1 + ax] = T[1 + ax] - 0.5 * self.q["g"] * ho * ho
        T = torch.stack(T[:self.nc])
        return (T if left else -T), (hL == 0) & (hR == 0)

    def linearize(self, U, off=True):
        """Residual, blocks [nb][nc][nc][ny][nx] (the diagonal one unregularized), isolated cells."""
        z, eps, nc = self.z, self.q["fd_eps"], self.nc
        own = self.side(U, z)
        pert = []
        for k in range(nc):
            Uk = U.clone()
            Uk[k] += eps
            pert.append(self.side(Uk, z))
        A = torch.zeros((1 + self.nf, nc, nc) + U.shape[1:], dtype=U.dtype, device=U.device)
        Rs, iso = torch.zeros_like(U), torch.ones_like(z, dtype=torch.bool)
        for f in range(self.nf):
            T0, dry = self.term(f, own, self.other(f, own, own))
            Rs += self.e[f] * T0
            iso &= dry
            inside = self.shift(torch.ones_like(z), f, 0.0)
            for k in range(nc):
                T, _ = self.term(f, pert[k], self.other(f, pert[k], own))
                A[0, :, k] += self.e[f] * ((T - T0) / eps)
                if off:
                    T, _ = self.term(f, own, self.other(f, own, pert[k]))
                    A[1 + f, :, k] = self.e[f] * ((T - T0) / eps) * inside
        return Rs, A, iso

    @staticmethod
    def solve(D, r):
        """D x = r in every cell, 0 where D is singular."""
        good = torch.linalg.det(D.permute(2, 3, 0, 1)) != 0
        eye = torch.eye(D.shape[0], dtype=D.dtype, device=D.device)
        M = torch.where(good[..., None, None], D.permute(2, 3, 0, 1), eye)
        x = torch.linalg.solve(M, torch.where(good[..., None], r.permute(1, 2, 0), 0.0)[..., None])
        return x[..., 0].permute(2, 0, 1)

    def regularize(self, A, Rs, U):
        """alpha ||R_i||_1 on the diagonal, and the rows of exactly dry cells."""
        nrm = Rs.abs().sum(0)
        for r in range(self.nc):
            A[0, r, r] += self.q["alpha"] * nrm
        Rs = Rs.clone()
        if self.q["dry_pin"]:
            dry = U[0] == 0
            for r in range(1, self.nc):
                A[:, r] = torch.where(dry, 0.0, A[:, r])
                A[0, r, r] = torch.where(dry, A[0, 0, 0], A[0, r, r])
                Rs[r] = torch.where(dry, 0.0, Rs[r])
        return Rs

    def blu(self, U):
        for c in (0, 1, 1, 0):
            Rs, A, _ = self.linearize(U, off=False)
            b = self.regularize(A, Rs, U)
            V = U - self.solve(A[0], b)
            V = torch.where(V[0] < self.q["h_eps"], 0.0, V)
            U = torch.where(self.colour(U.shape[1], U.shape[2], c), V, U)
        return U

    def assemble(self, U):
        Rs, A, iso = self.linearize(U)
        b = -self.regularize(A, Rs, U)
        b = torch.where(iso, 0.0, b)
        A = torch.where(iso, 0.0, A)
        for f in range(self.nf):
            A[1 + f] = torch.where(self.shift(iso.double(), f, 0.0) > 0, 0.0, A[1 + f])
        return Rs, A, b

    def product(self, A, x, first=0):
        y = torch.einsum("rcyx,cyx->ryx", A[0], x) if first == 0 else torch.zeros_like(x)
        for f in range(self.nf):
            y = y + torch.einsum("rcyx,cyx->ryx", A[1 + f], self.shift(x, f, 0.0))
        return y

    def coarsen(self, A):
        """Galerkin blocks of the next level: sums over the pairs of children."""
        out = torch.zeros(A.shape[:3] + (max(1, A.shape[3] // 2), A.shape[4] // 2), dtype=A.dtype,
                          device=A.device)
        rows = (0,) if self.nf == 2 else (0, 1)
        step = 1 if self.nf == 2 else 2
        for j in rows:
            for i in (0, 1):
                child = A[:, :, :, j::step, i::2]
                out[0] += child[0]
                for f in range(self.nf):
                    inner = (i == 1, i == 0, j == 1, j == 0)[f]
                    out[0 if inner else 1 + f] += child[1 + f]
        return out

    def total(self, r):
        r = r[:, :, 0::2] + r[:, :, 1::2]
        return r if self.nf == 2 else r[:, 0::2] + r[:, 1::2]

    def spread(self, x):
        x = x.repeat_interleave(2, 2)
        return x if self.nf == 2 else x.repeat_interleave(2, 1)

    def smooth(self, A, b, x, n):
        for _ in range(n):
            for c in (0, 1, 1, 0):
                y = self.solve(A[0], b - self.product(A, x, 1))
                x = torch.where(self.colour(x.shape[1], x.shape[2], c), y, x)
        return x

    def cycle(self, levels, l, b, x):
        q, A = self.q, levels[l]
        x = self.smooth(A, b, x, q["nu1"])
        if l + 1 == len(levels):
            x = self.smooth(A, b, x, q["nu_coarse"])
        else:
            bc = self.total(b - self.product(A, x))
            xc = torch.zeros_like(bc)
            for _ in range(1 if l == 0 else q["gamma"]):
                xc = self.cycle(levels, l + 1, bc, xc)
            x = x + self.spread(xc)
        return self.smooth(A, b, x, q["nu2"])

    def cycles(self, A, b, n):
        levels = [A]
        for _ in range(self.q["n_levels"]):
            levels.append(self.coarsen(levels[-1]))
        x = torch.zeros_like(b)
        for _ in range(n):
            x = self.cycle(levels, 0, b, x)
        return x

    def newton(self, U):
        """The Newton loop without the nested initial guess."""
        q = self.q
        U = torch.where(U[0] < q["h_eps"], 0.0, U)
        for _ in range(q["max_newton"]):
            for _ in range(q["blu_sweeps"]):
                U = self.blu(U)
            Rs, A, b = self.assemble(U)
            if not float(Rs.abs().sum()) >= TOL:
                break
            d = self.cycles(A, b, q["n_mg"])
            t, th = torch.full_like(U[0], q["tau"]), q["pos_theta"]
            if th > 0:
                cut = (d[0] < 0) & (U[0] + q["tau"] * d[0] < (1 - th) * U[0])
                t = torch.where(cut, th * U[0] / -d[0], t)
            U = U + t * d
            U = torch.where(U[0] < q["h_eps"], 0.0, U)
        return U


def exact(case, seed):
    kind, n = case["kind"], case["nx"] * case["ny"]
    if kind == "solve" and case["setting"] in ("bump", "smooth") and n <= 256:
        p = _problem(case, seed)
        return {"U": _Plain(p).newton(_dev(p.U0)), "steps": None, "sweeps": None, "pinned": None,
                "ok": None}
    if kind not in ("residual", "blu", "step"):
        return None             # hundreds of sweeps: too long written out like this
    p = _problem(case, seed)
    m, U = _Plain(p), _dev(p.U0)
    if kind == "residual":
        Rs, _, _ = m.linearize(U, off=False)
        return {"R": Rs, "norm": Rs.abs().sum().reshape(1)}
    if kind == "blu":
        return {"U": m.blu(U)}
    Rs, A, b = m.assemble(U)
    return {"R": Rs, "norm": float(Rs.abs().sum()), "dU": m.cycles(A, b, 3)}
