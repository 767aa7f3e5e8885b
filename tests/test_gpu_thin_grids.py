"""Grids a few cells wide: no more time than a square grid of as many cells
needs (half again, for the boundary cells and the timer), and the oracle's
results bit for bit.  Tiles and patches that suit square grids would leave
most of their lanes without a cell here.
"""
import numpy as np
import pytest

import oracle
from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def same(t, b, what):
    torch.cuda.synchronize()
    bad = t.cpu().numpy() != b
    assert not bad.any(), "%s: %d entries differ, first at %s" % (what, bad.sum(),
                                                                   np.argwhere(bad)[:3].tolist())


def still(nx, ny, **kw):
    z = np.zeros((ny, nx))
    U = np.zeros((3, ny, nx))
    U[0] = 1.0 + 0.01 * np.random.default_rng(1).uniform(-1, 1, (ny, nx))
    U[1] = 0.3
    return W.Problem("thin", 2, nx, ny, 0.0, 1.0, 0.0, 1.0, [W.wall()] * 4,
                     W.default_params(2, **kw), z, U)


def shortest(call, reps=5):
    """Milliseconds of the fastest of `reps` timings of ten calls each."""
    call()
    best = float("inf")
    for _ in range(reps):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 10)
    return best


def sweep_ms(nx, ny):
    from paper_1608_06721_amd import nmg
    p = still(nx, ny, n_levels=0)
    ctx = nmg.Context.from_problem(p)
    z, U = dev(p.z), dev(p.U0)
    ms = shortest(lambda: ctx.blu_sweep(z, U))
    ctx.close()
    return ms


@pytest.mark.parametrize("nx,ny", [(262144, 4), (4, 262144), (524288, 2), (131072, 8), (104858, 10),
                                   (65536, 16), (16, 65536), (128, 8192)])
def test_sweep_time(nx, ny):
    thin, square = sweep_ms(nx, ny), sweep_ms(1024, 1024)
    print("[thin sweep]", nx, ny, thin, square, flush=True)
    assert thin <= 1.5 * square


@pytest.mark.parametrize("nx,ny", [(131080, 4), (6, 131080)])
def test_sweep(nx, ny):
    from paper_1608_06721_amd import nmg
    z, U = W.random_state(2, nx, ny, 3)
    p = W.Problem("thin", 2, nx, ny, 0.0, 1.0, 0.0, 1.0,
                  [W.open_q(0.8, 0.0), W.open_h(1.1), W.wall(), W.wall(W.SLIP)],
                  W.default_params(2, n_levels=0), z, U)
    ctx = nmg.Context.from_problem(p)
    V = dev(U)
    ctx.blu_sweep(dev(z), V)
    same(V, oracle.blu_sweep(p, U), "U after a sweep")
    ctx.close()


def step_ms(nx, ny, **kw):
    """Assembly and three cycles from zero."""
    from paper_1608_06721_amd import nmg
    p = still(nx, ny, **kw)
    ctx = nmg.Context.from_problem(p)
    z, U = dev(p.z), dev(p.U0)
    x = torch.zeros_like(U)

    def call():
        ctx.assemble_residual_jacobian(z, U, want_norm=False)
        x.zero_()
        ctx.mg_vcycle(x, 3)
    ms = shortest(call, 3)
    ctx.close()
    return ms


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("nx,ny", [(2, 131072), (4, 65536), (6, 43692), (12, 21846), (131072, 2),
                                   (65536, 4), (32768, 8), (8192, 2), (2, 8192)])
def test_step_time(nx, ny, fp32, monkeypatch):
    """No coarse levels: runs of half sweeps against half sweeps one by one."""
    runs = step_ms(nx, ny, n_levels=0, inner_fp32=fp32)
    monkeypatch.setenv("NMG_FUSE", "1")
    single = step_ms(nx, ny, n_levels=0, inner_fp32=fp32)
    print("[thin step]", nx, ny, fp32, runs, single, flush=True)
    assert runs <= 1.5 * single


@pytest.mark.parametrize("coarse", ["0", "1024"])
@pytest.mark.parametrize("nx,ny,nl", [(2, 131080, 1), (8, 16384, 2), (16, 8200, 3), (34, 2048, 1),
                                      (40000, 2, 1), (2, 4096, 1)])
@pytest.mark.parametrize("fp32", [0, 1])
def test_cycles(nx, ny, nl, fp32, coarse, monkeypatch):
    from paper_1608_06721_amd import nmg
    monkeypatch.setenv("NMG_COARSE_CELLS", coarse)
    A, b = W.random_system(2, nx, ny, nx + ny)
    x0 = np.random.default_rng(3).uniform(-1, 1, b.shape)
    p = W.default_params(2, n_levels=nl, nu_coarse=3, inner_fp32=fp32)
    prob = W.Problem("thin", 2, nx, ny, 0, 1, 0, 1, [W.wall()] * 4, p, np.zeros((ny, nx)),
                     np.zeros_like(b))
    print("[thin cycles]", nx, ny, nl, fp32, flush=True)
    ctx = nmg.Context.from_problem(prob)
    ctx.load_system(dev(A), dev(b))
    x = dev(x0)
    ctx.mg_vcycle(x, 2)
    same(x, oracle.vcycles(A, b, x0, p, 2), "x after cycles")
    ctx.close()


def test_batch():
    """Instances under half a tile wide beside wider ones."""
    from paper_1608_06721_amd import nmg
    for sizes in ([(4, 4096)] * 20, [(8, 2048), (16, 1024), (64, 64), (2048, 8)] * 5):
        probs = [still(nx, ny, n_levels=1, max_newton=2) for nx, ny in sizes]
        for k, p in enumerate(probs):
            p.U0[1] += 0.01 * k
        batch = nmg.Batch(probs)
        Us = [dev(p.U0) for p in probs]
        batch.newton_mg_solve([dev(p.z) for p in probs], Us, 0.0)
        batch.close()
        for p, U in list(zip(probs, Us))[:6]:
            same(U, oracle.newton_solve(p, tol=0.0)[0], "U of %dx%d" % (p.nx, p.ny))
