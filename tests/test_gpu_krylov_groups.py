"""Krylov bases of the accelerated adjoint solve at the edges of the groups of
eight vectors that its products read at a time, on vectors that do not fill
their last block: the solution against the dense solve to 1e-9 of its largest entry
(a residual of 1e-13 and a condition number of about 65).
"""
import numpy as np
import pytest

import oracle
from blockmat import dense, unvec, vec
from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def slow(nx, ny):
    """Gentle flow without a coarse level: one smoothing step per cycle takes
    more steps than the bases below hold vectors."""
    r = np.random.default_rng(7)
    z = 0.02 * r.uniform(0, 1, (ny, nx))
    U = np.stack([1 + 0.02 * r.uniform(0, 1, (ny, nx)), np.full((ny, nx), 0.3),
                  0.01 * r.uniform(-1, 1, (ny, nx))])
    return W.Problem("slow", 2, nx, ny, 0.0, 2.0, 0.0, 1.0,
                     [W.open_q(0.3, 0.0), W.open_h(1.0), W.wall(), W.wall(W.SLIP)],
                     W.default_params(2, n_levels=0, nu1=1, nu_coarse=1), z, U)


@pytest.mark.parametrize("shape", [(36, 18), (48, 24)])
@pytest.mark.parametrize("krylov", [1, 7, 8, 9, 17])
def test_basis_sizes(shape, krylov):
    from paper_1608_06721_amd import nmg
    nx, ny = shape
    p = slow(nx, ny)
    z, U = p.z, p.U0.copy()
    ctx = nmg.Context.from_problem(p)
    g = np.random.default_rng(5).uniform(-1, 1, U.shape)
    lam, cyc, rel = ctx.adjoint_solve(dev(z), dev(U), dev(g), tol=1e-13, max_cycles=2000,
                                      krylov=krylov)
    torch.cuda.synchronize()
    print("[krylov]", shape, krylov, cyc, rel, flush=True)
    assert rel <= 1e-13
    A, _, _ = oracle.assemble(p, U)
    ref = unvec(np.linalg.solve(dense(oracle.transpose_blocks(A)), vec(g)), 3, ny, nx)
    assert krylov < 8 or cyc > krylov, cyc      # the basis was filled
    np.testing.assert_allclose(lam.cpu().numpy(), ref, rtol=0, atol=1e-9 * np.abs(ref).max())
    ctx.close()
