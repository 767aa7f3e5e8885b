"""Runs of half sweeps on the wide tiles of large levels (32x16, with a
restriction 28x16 in FP64 and 32x16 or 48x16 in FP32) against the oracle, bit
for bit: level sizes just above 2^16 and 2^17 cells, whole tiles, one pair of
cells past them and thin grids, run lengths on both sides of the shortest run,
single and batched (the batch's finest level in runs as well).
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


GRIDS = [(256, 258), (288, 288), (282, 242), (8, 8200), (11000, 6), (512, 256), (336, 400),
         (386, 354), (514, 514)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("nus", [(2, 2), (1, 3), (3, 1)])
@pytest.mark.parametrize("fp32", [0, 1])
def test_cycles(grid, nus, fp32, monkeypatch):
    from paper_1608_06721_amd import nmg
    nx, ny = grid
    print("[wide runs]", grid, nus, fp32, flush=True)
    monkeypatch.setenv("NMG_COARSE_CELLS", "0")
    A, b = W.random_system(2, nx, ny, nx + ny)
    x0 = np.random.default_rng(5).uniform(-1, 1, b.shape)
    p = W.default_params(2, n_levels=1, nu1=nus[0], nu2=nus[1], nu_coarse=2, inner_fp32=fp32)
    prob = W.Problem("runs", 2, nx, ny, 0, 1, 0, 1, [W.wall()] * 4, p, np.zeros((ny, nx)),
                     np.zeros_like(b))
    ctx = nmg.Context.from_problem(prob)
    ctx.load_system(dev(A), dev(b))
    x = dev(x0)
    ctx.mg_vcycle(x, 2)
    same(x, oracle.vcycles(A, b, x0, p, 2), "x after cycles")
    if not fp32:        # the restricted right-hand side of the last cycle
        y = oracle.sgs(A, b, oracle.vcycles(A, b, x0, p, 1), nus[0], order=W.REDBLACK)
        same(ctx.get_system(1)[1], oracle.restrict(A, b, y), "restricted residual")
    ctx.close()


@pytest.mark.parametrize("n_mg", [1, 2])
@pytest.mark.parametrize("fp32", [0, 1])
def test_batch_finest_level(n_mg, fp32):
    from paper_1608_06721_amd import nmg
    probs = W.batch_channels(3, sizes=(256, 288, 320), seed=4, n_levels=3, gamma=2, n_mg=n_mg,
                             inner_fp32=fp32, max_newton=2)
    batch = nmg.Batch(probs)
    for _ in range(2):
        Us = [dev(p.U0) for p in probs]
        batch.newton_mg_solve([dev(p.z) for p in probs], Us, 0.0)
        for p, U in zip(probs, Us):
            same(U, oracle.newton_solve(p, tol=0.0)[0], p.name)
    batch.close()
