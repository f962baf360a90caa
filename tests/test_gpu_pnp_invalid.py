"""Invalid hypotheses: scored -1, whatever they are paired with, and not counted over the matches.

A workgroup takes two hypotheses; any of the two, both or none may be invalid (a sample index out
of range).  A valid one's score may not depend on its neighbour: it is that of the same samples in
another pairing and with every hypothesis valid.  The cost of an invalid one is that of finding
it so: with every hypothesis invalid a call takes less than half of a call's time (it streams no
matches; at the sizes here the other kernels take a few per cent).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402
from paper_2507_03737_amd.tracking import PnpConfig, pnp_ransac  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu

CAM = Camera(640, 480, 500.0, 500.0, 320.0, 240.0)


def problem(n, seed):
    rng = np.random.default_rng(seed)
    X = np.stack([rng.uniform(-2, 2, n), rng.uniform(-2, 2, n), rng.uniform(2, 6, n)])
    uv = np.stack([500 * X[0] / X[2] + 320, 500 * X[1] / X[2] + 240]) + rng.normal(0, 0.5, (2, n))
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    return f32(X), f32(uv), rng


def scores_of(X, uv, samples):
    cfg = PnpConfig(n_hypotheses=len(samples), threshold=2.0, iterations=1, rounds=1)
    return pnp_ransac(X, uv, CAM, torch.from_numpy(samples.astype(np.int32)).cuda(), cfg)[3].cpu().numpy()


@pytest.mark.parametrize("hyps", [1, 2, 3, 64, 65])
@pytest.mark.parametrize("n", [6, 511, 3000])
def test_scores_beside_invalid_hypotheses(n, hyps):
    U.log(f"[gpu] pnp invalid hypotheses n {n} hypotheses {hyps}")
    X, uv, rng = problem(n, n + hyps)
    samples = np.stack([rng.permutation(n)[:6] for _ in range(hyps)])
    want = scores_of(X, uv, samples)
    assert np.all(want >= 0)
    for bad in (rng.random(hyps) < 0.5, np.arange(hyps) % 2 == 0, np.arange(hyps) % 2 == 1, np.ones(hyps, bool)):
        mixed = samples.copy()
        mixed[bad, rng.integers(0, 6)] = rng.choice([-1, n])
        assert np.array_equal(scores_of(X, uv, mixed), np.where(bad, -1, want))
    shifted = np.concatenate([samples[-1:], samples[:-1]])
    assert np.array_equal(scores_of(X, uv, shifted), np.roll(want, 1))


def test_invalid_hypotheses_cost_little():
    U.log("[gpu] pnp time of invalid hypotheses")
    n, hyps = 1 << 19, 2048
    X, uv, rng = problem(n, 1)
    cfg, ctx, times = PnpConfig(n_hypotheses=hyps, iterations=0, rounds=0), binding.Context(), {}
    for name, first in (("valid", 0), ("invalid", -1)):
        samples = torch.from_numpy(rng.integers(0, n, (hyps, 6)).astype(np.int32)).cuda()
        if first < 0:
            samples[:, 0] = first
        runs = []
        for _ in range(7):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            pnp_ransac(X, uv, CAM, samples, cfg, ctx=ctx)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        times[name] = float(np.median(runs))
    assert times["invalid"] < 0.5 * times["valid"], times
