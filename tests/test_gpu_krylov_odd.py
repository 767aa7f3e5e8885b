"""The accelerated adjoint solve on odd widths: the colour-split vectors then
have a slot without a cell in some or every row, which the sums of the Krylov
basis run over.  Two restart lengths on one context (its vectors are freed and
allocated again) in memory that held NaN before: the solution against the
dense solve to 1e-9 of its largest entry (a residual of 1e-13 and a condition
number below 100), the same number of cycles whatever the memory held.
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


def gentle(dim, nx, ny):
    r = np.random.default_rng(7)
    z = 0.02 * r.uniform(0, 1, (ny, nx))
    U = np.stack([1 + 0.02 * r.uniform(0, 1, (ny, nx)), np.full((ny, nx), 0.3),
                  0.01 * r.uniform(-1, 1, (ny, nx))][:dim + 1])
    return W.Problem("gentle", dim, nx, ny, 0.0, 2.0, 0.0, 1.0,
                     [W.open_q(0.3, 0.0), W.open_h(1.0), W.wall(), W.wall(W.SLIP)],
                     W.default_params(dim, n_levels=0, nu1=1, nu_coarse=1), z, U)


def dirty():
    """Leave NaN in the device memory that the next allocations get."""
    for n in (1 << 10, 1 << 14, 1 << 16, 1 << 18, 1 << 20, 1 << 22):
        keep = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
                for _ in range(8)]
    torch.cuda.synchronize()
    del keep
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dim,nx,ny", [(2, 35, 17), (2, 5, 32), (2, 34, 17), (1, 33, 1)])
def test_slots_without_cells(dim, nx, ny):
    from paper_1608_06721_amd import nmg
    p = gentle(dim, nx, ny)
    z, U = dev(p.z), dev(p.U0)
    g = np.random.default_rng(5).uniform(-1, 1, p.U0.shape)
    A, _, _ = oracle.assemble(p, p.U0)
    ref = unvec(np.linalg.solve(dense(oracle.transpose_blocks(A)), vec(g)), dim + 1, ny, nx)
    cycles = {}
    for again in range(2):
        ctx = nmg.Context.from_problem(p)
        for m in (9, 17):
            dirty()
            lam, cyc, rel = ctx.adjoint_solve(z, U, dev(g), tol=1e-13, max_cycles=2000, krylov=m)
            torch.cuda.synchronize()
            print("[krylov odd]", dim, nx, ny, m, cyc, rel, flush=True)
            assert rel <= 5e-12 and cycles.setdefault(m, cyc) == cyc
            np.testing.assert_allclose(lam.cpu().numpy(), ref, rtol=0,
                                       atol=1e-9 * np.abs(ref).max())
        ctx.close()
