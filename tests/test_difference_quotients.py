"""The forward-difference quotients of the HIP kernels: (Tk - T0) / eps is
formed from a reciprocal of eps that the host splits in two, and has to be
the correctly rounded quotient for every difference and step.

On the CPU the recipe itself, with exactly rounded operations, against the
division; on the GPU whole assemblies and sweeps against the oracle, bit for
bit, with steps whose reciprocals round well and badly, every flux, and
states whose differences span the exponent range.
"""
import math
import sys
from fractions import Fraction

import numpy as np
import pytest

import oracle
from paper_1608_06721_amd import workloads as W

STEPS = [1e-8, 1e-6, 3e-7, 1.0 / 3.0, 2.0 ** -27, 0.7e-9, 1.9999999e-5]


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))      # one rounding


def quotient(a, eps):
    """The recipe of the kernels' fd_quotient, without the factor |e|."""
    rh = 1.0 / eps
    rl = fma(-rh, eps, 1.0) / eps
    q0 = fma(a, rh, a * rl)
    return fma(fma(-q0, eps, a), rh, q0)


def differences(rng, eps):
    out = [0.0, 1.0, -1.0, 2.0 ** -960, 1e290, np.nextafter(1.0, 2), np.nextafter(2.0, 1)]
    m = rng.integers(2 ** 52, 2 ** 53, 300)
    out += [math.ldexp(float(v), int(e)) for v, e in zip(m, rng.integers(-900, 800, 300))]
    # quotients next to a rounding boundary: a = the double nearest (q + ulp / 2) eps
    for q in rng.uniform(0.5, 2.0, 300):
        mid = (Fraction(float(q)) + Fraction(float(np.nextafter(q, 4)))) / 2
        a = float(mid * Fraction(eps))
        out += [a, float(np.nextafter(a, 0)), float(np.nextafter(a, 4))]
    return out


@pytest.mark.parametrize("eps", STEPS)
def test_quotient_is_the_division(eps):
    for a in differences(np.random.default_rng(7), eps):
        assert quotient(a, eps) == a / eps, (a, eps)


torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def same(t, b, what):
    torch.cuda.synchronize()
    a = t.cpu().numpy()
    bad = ~((a == b) | (np.isnan(a) & np.isnan(b)))
    assert not bad.any(), "%s: %d entries differ, first at %s" % (what, bad.sum(),
                                                                   np.argwhere(bad)[:3].tolist())


def state(dim, kind):
    nx, ny = (33, 1) if dim == 1 else (21, 13)
    z, U = W.random_state(dim, nx, ny, 31)
    if kind == "tiny_momentum":
        U[1:] *= 1e-270
    elif kind == "thin":
        U[0] *= 1e-5
        z[:] = 0.25
    elif kind == "huge":
        U *= 1e60
    elif kind == "infinite":
        U[0, 0, 3] = np.inf
        U[1, 0, 7] = np.nan
    return nx, ny, z, U


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "tiny_momentum", "thin", "huge", "infinite"])
@pytest.mark.parametrize("dim,flux", [(1, W.HLL), (1, W.LLF), (2, W.HLL), (2, W.LLF), (2, W.HLLC)])
def test_assembly_and_sweep(dim, flux, kind, monkeypatch):
    from paper_1608_06721_amd import nmg
    nx, ny, z, U = state(dim, kind)
    bc = [W.open_q(0.8, 0.0), W.open_h(1.1), W.wall(), W.wall(W.SLIP)]
    for eps in STEPS[:4]:
        prm = W.default_params(dim, flux=flux, n_levels=0, fd_eps=eps)
        prob = W.Problem("q", dim, nx, ny, 0.0, nx / 4.0, 0.0, ny / 4.0 if dim == 2 else 1.0, bc,
                         prm, z, U)
        print("[quotients]", dim, flux, kind, eps, flush=True)
        sys.stdout.flush()
        Ao, bo, _ = oracle.assemble(prob, U)
        Uo = oracle.blu_sweep(prob, U)
        for lanes in ("1", "4", "16"):
            monkeypatch.setenv("NMG_BLU_LANES", lanes)
            ctx = nmg.Context.from_problem(prob)
            if lanes == "1":
                ctx.assemble_residual_jacobian(dev(z), dev(U), want_norm=False)
                A, b = ctx.get_system(0)
                same(A, Ao, "A")
                same(b, bo, "b")
            V = dev(U)
            ctx.blu_sweep(dev(z), V)
            same(V, Uo, "U after a sweep, %s lanes" % lanes)
            ctx.close()


# Inflow sides on every side of the grid, in both slot orders and with waves
# that are full, ragged and nearly empty: the celerities of a wave's boundary
# cells are formed together.
@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(2, 2), (5, 3), (130, 66), (63, 129), (1030, 520)])
@pytest.mark.parametrize("qn", [0.8, 1e-3, 1e70])
def test_inflow_sides(nx, ny, qn, monkeypatch):
    from paper_1608_06721_amd import nmg
    z, U = W.random_state(2, nx, ny, 5)
    for bc in ([W.open_q(qn, 0.1), W.open_h(1.1), W.open_q(qn), W.open_q(qn, 0.0)],
               [W.open_h(1.0), W.open_q(qn), W.wall(W.SLIP), (W.OPEN, 0.9, qn, 0.2)]):
        prob = W.Problem("in", 2, nx, ny, 0.0, 5.0, 0.0, 3.0, bc, W.default_params(2, n_levels=0),
                         z, U)
        print("[inflow]", nx, ny, qn, flush=True)
        monkeypatch.setenv("NMG_BLU_LANES", "1")
        ctx = nmg.Context.from_problem(prob)
        V = dev(U)
        ctx.blu_sweep(dev(z), V)
        same(V, oracle.blu_sweep(prob, U), "U after a sweep")
        ctx.assemble_residual_jacobian(dev(z), dev(U), want_norm=False)
        same(ctx.get_system(0)[0], oracle.assemble(prob, U)[0], "A")
        ctx.close()
