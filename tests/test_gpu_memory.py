"""Device memory of a context and of a batch: what is kept besides the
hierarchy, and contexts where there is no room for it: the same results from
single launches.
"""
import numpy as np
import pytest

import oracle
from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 2048
MB = 1 << 20


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def flow(n, steps=1, **kw):
    z = 0.1 * np.sin(np.arange(n) / n * 9)[None, :] * np.cos(np.arange(n) / n * 5)[:, None]
    U = np.zeros((3, n, n))
    U[0] = 1.0 - z
    U[1] = 0.5
    return W.Problem("memory", 2, n, n, 0.0, 10.0, 0.0, 2.0,
                     [W.open_q(1.0, 0.0), W.open_h(1.0), W.wall(), W.wall()],
                     W.default_params(2, n_levels=6, n_mg=2, max_newton=steps, **kw), z, U)


def hierarchy_bytes(n, levels):
    """Blocks, b and x of every level, and the kept iterate."""
    return sum(8 * (45 + 6) * (n >> l) ** 2 for l in range(levels + 1)) + 8 * 3 * n * n


def context(nmg, p, monkeypatch=None, fuse=None):
    if fuse is not None:
        monkeypatch.setenv("NMG_FUSE", fuse)
    ctx = nmg.Context.from_problem(p)
    if fuse is not None:
        monkeypatch.delenv("NMG_FUSE")
    return ctx


def test_footprint(monkeypatch):
    """Runs of half sweeps keep a second x (3 of 54 doubles a cell with the kept
    iterate, 6 %) and nothing more; single launches half of one (the residual
    planes)."""
    from paper_1608_06721_amd import nmg
    p = flow(N)
    context(nmg, p).close()                 # (what the first use of the GPU takes)
    base = hierarchy_bytes(N, 6)
    x = 8 * 3 * N * N
    for fuse, most in ((None, 1.34 * x), ("1", 0.51 * x)):
        before = free()
        ctx = context(nmg, p, monkeypatch, fuse)
        used = before - free()
        ctx.close()
        print("[memory]", fuse, used / MB, base / MB, most / MB, flush=True)
        assert used <= base + most + 32 * MB


def fill(leave):
    """Tensors that leave about `leave` bytes of the GPU's memory free."""
    out = []
    while free() > leave + 2 * MB:
        out.append(torch.empty(min(free() - leave, 16 << 30), dtype=torch.uint8, device="cuda"))
    return out


def solve(nmg, p, make):
    z, U = dev(p.z), dev(p.U0)
    ctx = make()
    ctx.newton_mg_solve(z, U, 0.0)
    torch.cuda.synchronize()
    out = U.cpu().numpy()
    ctx.close()
    return out


def test_no_room_for_runs(monkeypatch):
    from paper_1608_06721_amd import nmg
    p = flow(N)
    want = solve(nmg, p, lambda: nmg.Context.from_problem(p))
    z, U = dev(p.z), dev(p.U0)
    before = free()
    ctx = context(nmg, p, monkeypatch, "1")
    single = before - free()
    ctx.close()
    # less than the second x buffers (134 MB) and than the residual planes (50 MB)
    keep = fill(single - 50 * MB + 40 * MB)
    print("[memory] single", single / MB, "free", free() / MB, flush=True)
    ctx = nmg.Context.from_problem(p)
    ctx.newton_mg_solve(z, U, 0.0)
    torch.cuda.synchronize()
    left = free()
    got = U.cpu().numpy()
    ctx.close()
    del keep
    free()
    print("[memory] left", left / MB, flush=True)
    assert left < 100 * MB
    assert np.array_equal(got, want)


def test_no_room_for_a_batch(monkeypatch):
    from paper_1608_06721_amd import nmg
    probs = [flow(1024), flow(512)]
    zs, U0s, Us = ([dev(a) for a in x] for x in
                   ([p.z for p in probs], [p.U0 for p in probs], [p.U0 for p in probs]))

    def run():
        for U, U0 in zip(Us, U0s):
            U.copy_(U0)
        b = nmg.Batch(probs)
        b.newton_mg_solve(zs, Us, 0.0)
        torch.cuda.synchronize()
        left = free()
        b.close()
        return left, [U.cpu().numpy() for U in Us]

    _, want = run()
    before = free()
    monkeypatch.setenv("NMG_FUSE", "1")
    b = nmg.Batch(probs)
    monkeypatch.delenv("NMG_FUSE")
    single = before - free()
    b.close()
    # less than the second x buffers (40 MB) and than the residual planes (15 MB)
    keep = fill(single - 15 * MB + 10 * MB)
    left, got = run()
    del keep
    free()
    print("[memory] batch left", left / MB, flush=True)
    assert left < 30 * MB
    assert all(np.array_equal(a, c) for a, c in zip(got, want))


@pytest.mark.parametrize("krylov,captured", [(0, False), (4, False), (0, True)])
def test_adjoint_takes_the_runs_memory(krylov, captured):
    """The transposed matrix (1.5 GB) or the Krylov vectors (0.8 GB) fit only
    without the second x (134 MB): given back, unless a graph may use it."""
    from paper_1608_06721_amd import nmg
    p = flow(N)
    z, U = dev(p.z), dev(p.U0)
    g = torch.ones_like(U)
    s = torch.cuda.Stream()
    out = {}
    for full in (False, True):
        with torch.cuda.stream(s):
            ctx = nmg.Context.from_problem(p)
            lam, x = torch.zeros_like(U), torch.zeros_like(U)
            ctx.assemble_residual_jacobian(z, U, want_norm=False)
            ctx.mg_vcycle(x, 1)
            if captured:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=s):
                    ctx.mg_vcycle(x, 1)
            s.synchronize()
            keep = []
            if full:
                need = 8 * 45 * N * N + (8 * 3 * N * N * 8 if krylov else 0)
                keep = fill(need - 70 * MB)
            try:
                ctx.adjoint_solve(z, U, g, lam, tol=0.0, max_cycles=2, krylov=krylov)
                s.synchronize()
                x.zero_()
                ctx.mg_vcycle(x, 1)         # (of the adjoint's system)
                s.synchronize()
                out[full] = lam.cpu().numpy(), x.cpu().numpy()
            except nmg.NMGError as e:
                assert full and captured, e
                s.synchronize()
                out[full] = out[False]
            else:
                assert not (full and captured)
            del keep
            free()
            if captured:
                graph.replay()
                s.synchronize()
                del graph
            ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(out[False], out[True]))
