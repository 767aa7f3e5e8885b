"""BLU-SGS sweeps in one launch (tiles of 4 x 2 and 4 x 4 cells) against the
oracle, bit for bit: whole Newton steps and Step 1 on meshes of one cell of a
tile up to the largest that runs this way and the first that does not, with
every flux and boundary kind, with threshold stops, caps of either parity (the
state ends in either of two buffers) and graph replays.
"""
import numpy as np
import pytest

import oracle
from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def solve(prob, repeats=1):
    from paper_1608_06721_amd import nmg
    ctx = nmg.Context.from_problem(prob)
    Uo, so = oracle.newton_solve(prob, tol=0.0)
    for _ in range(repeats):
        U = dev(prob.U0)
        st = ctx.newton_mg_solve(dev(prob.z), U, 0.0)
        torch.cuda.synchronize()
        assert st["newton_steps"] == so["newton_steps"]
        bad = U.cpu().numpy() != Uo
        assert not bad.any(), "%d entries differ, first at %s" % (bad.sum(),
                                                                  np.argwhere(bad)[:3].tolist())
    ctx.close()
    return st


@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 5), (4, 2), (5, 3), (7, 9), (33, 31), (64, 32),
                                   (66, 32), (64, 64), (66, 64)])
@pytest.mark.parametrize("flux", [W.HLL, W.LLF, W.HLLC])
@pytest.mark.parametrize("sweeps", [1, 2])
def test_newton_steps(nx, ny, flux, sweeps):
    z, U = W.random_state(2, nx, ny, nx)
    bc = [W.open_q(0.8, 0.0), W.open_h(1.1), W.wall(), W.wall(W.SLIP)]
    p = W.default_params(2, flux=flux, n_levels=0, blu_sweeps=sweeps, max_newton=2)
    print("[sweep tiles]", nx, ny, flux, sweeps, flush=True)
    solve(W.Problem("t", 2, nx, ny, 0.0, 5.0, 0.0, 3.0, bc, p, z, U))


@pytest.mark.parametrize("cap", [0, 1, 2, 3, 62, 63, 64, 65, 129, 1000])
@pytest.mark.parametrize("nx,ny,nl", [(64, 32, 3), (128, 128, 2), (40, 72, 2)])
def test_step1(nx, ny, nl, cap):
    prob = W.dry_hill(nx, ny, n_levels=nl, eps_p=0.2, init_max_sweeps=cap, max_newton=2)
    print("[sweep tiles] step 1", nx, ny, nl, cap, flush=True)
    st = solve(prob, repeats=2)
    so = oracle.newton_solve(prob, tol=0.0)[1]
    assert st["init_sweeps"] == so["init_sweeps"]
