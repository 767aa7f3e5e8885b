"""A caller's HIP graph of an assembly, a BLU-SGS sweep and cycles: runs of half
sweeps let a level's two buffers change places, so a replay starts from
buffers that the context may have left the other way round.  Every replay, with
eager calls on other data between them, equals the eager result.
"""
import numpy as np
import pytest

import oracle
from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("dim,nx,ny,levels,nus,coarse", [
    (2, 96, 64, 3, (2, 2), "1024"), (2, 96, 64, 3, (2, 2), "0"), (2, 40, 24, 2, (3, 1), "0"),
    (2, 320, 256, 2, (2, 2), "1024"), (1, 256, 1, 3, (2, 2), "1024")])
def test_replays(dim, nx, ny, levels, nus, coarse, monkeypatch):
    from paper_1608_06721_amd import nmg
    monkeypatch.setenv("NMG_COARSE_CELLS", coarse)
    mk = (lambda k: W.random_state(dim, nx, ny, k))
    z, U0 = mk(1)
    p = W.Problem("graph", dim, nx, ny, 0.0, 3.0, 0.0, 2.0,
                  [W.open_q(0.8, 0.0), W.open_h(1.1), W.wall(), W.wall(W.SLIP)],
                  W.default_params(dim, n_levels=levels, nu1=nus[0], nu2=nus[1], nu_coarse=2), z, U0)
    want = {}
    for k in (1, 2, 3):
        U = oracle.blu_sweep(p, mk(k)[1])
        A, b, _ = oracle.assemble(p, U)
        want[k] = U, oracle.vcycles(A, b, np.zeros_like(b), p.params, 3)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = nmg.Context.from_problem(p)
        zd, U, x = dev(z), dev(U0), dev(np.zeros_like(U0))

        def call(U, x):
            ctx.blu_sweep(zd, U)
            ctx.assemble_residual_jacobian(zd, U, want_norm=False)
            x.zero_()
            ctx.mg_vcycle(x, 3)

        def check(k, U, x, what):
            s.synchronize()
            assert np.array_equal(U.cpu().numpy(), want[k][0]), what
            assert np.array_equal(x.cpu().numpy(), want[k][1]), what

        call(U, x)
        check(1, U, x, "eager")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call(U, x)
        V, y = dev(U0), dev(np.zeros_like(U0))
        for n, k in enumerate((2, 3, 1, 1, 2, 3)):
            U.copy_(dev(mk(k)[1]))
            g.replay()
            check(k, U, x, "replay %d" % n)
            if n % 2 == 0:
                V.copy_(dev(mk(3)[1]))
                call(V, y)
                check(3, V, y, "eager after replay %d" % n)
            else:
                ctx.mg_vcycle(y, 1)
        s.synchronize()
        ctx.close()
