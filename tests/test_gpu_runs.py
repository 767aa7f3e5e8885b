"""Runs of half sweeps on tiles (one launch for up to five half sweeps and the
restriction that follows) against the oracle, bit for bit: grids one tile
wide, at the edges of tiles and one pair of cells past them, for every tile
width that a level's size selects, with even and uneven run lengths, from
zero, stored and prolonged corrections, single and batched.
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


# level-0 size, levels: tiles of 8 (up to 2^13 cells), 16 (2^15), 32 (2^17)
# and 16 again (FP64, 2^18) cells by 8 rows
GRIDS = [(2, 2, 0), (4, 4, 1), (8, 8, 1), (10, 8, 1), (16, 18, 1), (14, 34, 1), (132, 68, 2),
         (144, 128, 1), (146, 130, 1), (260, 132, 2), (256, 136, 1), (322, 404, 1), (516, 260, 2)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("nus", [(2, 2, 3), (3, 1, 2), (1, 0, 1)])
@pytest.mark.parametrize("fp32", [0, 1])
def test_cycles(grid, nus, fp32, monkeypatch):
    from paper_1608_06721_amd import nmg
    nx, ny, nl = grid
    print("[runs]", grid, nus, fp32, flush=True)
    monkeypatch.setenv("NMG_COARSE_CELLS", "0")
    A, b = W.random_system(2, nx, ny, nx + ny)
    x0 = np.random.default_rng(3).uniform(-1, 1, b.shape)
    p = W.default_params(2, n_levels=nl, nu1=nus[0], nu2=nus[1], nu_coarse=nus[2], gamma=2,
                         inner_fp32=fp32)
    prob = W.Problem("runs", 2, nx, ny, 0, 1, 0, 1, [W.wall()] * 4, p, np.zeros((ny, nx)),
                     np.zeros_like(b))
    ctx = nmg.Context.from_problem(prob)
    ctx.load_system(dev(A), dev(b))
    x = dev(x0)
    ctx.mg_vcycle(x, 2)
    same(x, oracle.vcycles(A, b, x0, p, 2), "x after cycles")
    if nl:      # the restricted right-hand side of the last cycle
        y = oracle.vcycles(A, b, x0, p, 1)
        if nus[0]:
            y = oracle.sgs(A, b, y, nus[0], order=W.REDBLACK) if not fp32 else None
        if not fp32:
            same(ctx.get_system(1)[1], oracle.restrict(A, b, y), "restricted residual")
    ctx.close()


@pytest.mark.parametrize("coarse", ["0", "1024"])
@pytest.mark.parametrize("fp32", [0, 1])
def test_batch(coarse, fp32, monkeypatch):
    """Uneven instances whose launched coarse levels run on tiles, over
    several Newton steps (the levels' two buffers change places)."""
    from paper_1608_06721_amd import nmg
    monkeypatch.setenv("NMG_COARSE_CELLS", coarse)
    probs = W.batch_channels(4, sizes=(96, 128, 160), seed=21, n_levels=3, gamma=2, nu1=1,
                             inner_fp32=fp32, max_newton=4)
    batch = nmg.Batch(probs)
    for _ in range(2):
        Us = [dev(p.U0) for p in probs]
        batch.newton_mg_solve([dev(p.z) for p in probs], Us, 0.0)
        for p, U in zip(probs, Us):
            same(U, oracle.newton_solve(p, tol=0.0)[0], p.name)
    batch.close()
