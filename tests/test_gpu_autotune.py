"""The batch autotuner tunes what the batch launches: levels smoothed in runs
keep the default tile length, those whose half sweeps are launched one by one
get one of the four, and the tuned tiles change no result.
"""
import numpy as np
import pytest

from paper_1608_06721_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def solve(nmg, probs, tuned):
    b = nmg.Batch(probs)
    tiles = None
    if tuned:
        tiles = [b.autotune(reps=3) for _ in range(4)]
    Us = [dev(p.U0) for p in probs]
    b.newton_mg_solve([dev(p.z) for p in probs], Us, 0.0)
    torch.cuda.synchronize()
    b.close()
    return tiles, [U.cpu().numpy() for U in Us]


# launched: the levels whose half sweeps are launched one by one (three FP64
# iterations on a level of more than 2^16 cells are, where the first colour is
# elided: six half sweeps make two runs of three, too short for such a level)
@pytest.mark.parametrize("fuse,nu,fp32,launched", [
    ("5", (2, 2), 0, ()), ("5", (2, 2), 1, ()), ("5", (3, 2), 0, (0,)), ("5", (3, 3), 1, ()), ("1", (2, 2), 0, (0, 1)),
    ("1", (1, 1), 1, (0, 1)), ("5", (1, 1), 0, (0,)), ("2", (2, 2), 1, (0, 1))])
def test_tuned_levels(fuse, nu, fp32, launched, monkeypatch):
    from paper_1608_06721_amd import nmg
    monkeypatch.setenv("NMG_FUSE", fuse)
    monkeypatch.setenv("NMG_COARSE_CELLS", "1024")
    # 5 grids of 96x160 to 160x160: more than 2^16 cells on level 0, less on level 1,
    # level 2 (up to 40x40) launched too, level 3 in the coarse kernel
    probs = [W.channel(nx, 160, seed=W.BATCH_SEED + k, n_levels=3, nu1=nu[0], nu2=nu[1],
                       inner_fp32=fp32, max_newton=3) for k, nx in enumerate((96, 128, 160, 160, 96))]
    tiles, tuned = solve(nmg, probs, True)
    print("[autotune]", fuse, nu, fp32, tiles, flush=True)
    for t in tiles:
        assert len(t) == 4 and all(v in (64, 128, 256, 512) for v in t)
        for l in range(4):
            if not launched or (l not in launched and (l > 2 or fuse == "5")):
                assert t[l] == 256
    _, plain = solve(nmg, probs, False)
    for p, a, b in zip(probs, tuned, plain):
        assert np.array_equal(a, b), p.name


def test_one_dimension():
    from paper_1608_06721_amd import nmg
    probs = [W.smooth_1d(n, n_levels=2, max_newton=3) for n in (8192, 16384)]
    tiles, tuned = solve(nmg, probs, True)
    print("[autotune]", tiles, flush=True)
    assert all(v in (64, 128, 256, 512) for t in tiles for v in t)
    _, plain = solve(nmg, probs, False)
    assert all(np.array_equal(a, b) for a, b in zip(tuned, plain))
