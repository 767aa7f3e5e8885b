"""Galerkin products of large 1D levels, formed by rows: bit for bit those of
the oracle in either precision, single and batched, at the size where rows
replace entries, and in the time of a copy of as many bytes or half again.
"""
import numpy as np
import pytest

import oracle
from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def line(n, levels, **kw):
    return W.smooth_1d(n, n_levels=levels, **kw)


def same(t, b, what):
    torch.cuda.synchronize()
    bad = t.cpu().numpy() != b
    assert not bad.any(), "%s: %d entries differ, first at %s" % (what, bad.sum(),
                                                                   np.argwhere(bad)[:3].tolist())


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("n", [32764, 32768, 32772, 131076])
def test_levels(n, fp32):
    from paper_1608_06721_amd import nmg
    p = line(n, 2, inner_fp32=fp32)
    A, b = W.random_system(1, n, 1, 7)
    if fp32:
        A = A.astype(np.float32).astype(np.float64)
    print("[galerkin 1d]", n, fp32, flush=True)
    ctx = nmg.Context.from_problem(p)
    ctx.load_system(dev(A), dev(b))
    for l in (1, 2):
        if fp32:            # sums of floats, in the oracle's order
            f = [A[k].astype(np.float32) for k in range(3)]
            L, R = [g[..., 0::2] for g in f], [g[..., 1::2] for g in f]
            D = ((np.float32(0) + L[0] + L[2]) + R[1]) + R[0]
            w, e = np.float32(0) + L[1], np.float32(0) + R[2]
            w[..., 0] = 0
            e[..., -1] = 0
            A = np.stack([D, w, e]).astype(np.float64)
        else:
            A = oracle.galerkin(A)
        same(ctx.get_system(l, want_b=False)[0], A, "A of level %d" % l)
    ctx.close()


def test_batch():
    from paper_1608_06721_amd import nmg
    probs = [line(n, 2, max_newton=2) for n in (32768, 16384, 49156)]
    batch = nmg.Batch(probs)
    Us = [dev(p.U0) for p in probs]
    batch.newton_mg_solve([dev(p.z) for p in probs], Us, 0.0)
    batch.close()
    for p, U in zip(probs, Us):
        same(U, oracle.newton_solve(p, tol=0.0)[0], p.name)


def shortest(call, reps=5):
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


def test_rate():
    from paper_1608_06721_amd import nmg
    n, ms = 1 << 22, []
    for levels in (0, 1):
        p = line(n, levels)
        ctx = nmg.Context.from_problem(p)
        z, U = dev(p.z), dev(p.U0)
        ms.append(shortest(lambda: ctx.assemble_residual_jacobian(z, U, want_norm=False)))
        ctx.close()
    src = torch.empty(9 * n, dtype=torch.float64, device="cuda")    # 12 n read, 6 n written
    dst = torch.empty_like(src)
    copy = shortest(lambda: dst.copy_(src))
    print("[galerkin 1d rate]", ms, copy, flush=True)
    assert ms[1] - ms[0] <= 1.5 * copy       # (by entries 2.1)
