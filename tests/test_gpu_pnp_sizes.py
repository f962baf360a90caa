"""RANSAC + PnP at the sizes where its kernels change: as few matches as a sample, around a
workgroup's 256 lanes and beyond the 256 workgroups of a step, odd numbers of hypotheses, and
no refinement at all, against the float64 oracle on the same float32 inputs.

The pose minimises the same sums in float64, in another order: its bound is the one that the
oracle comparison of the usual sizes uses, 1e-9.  Samples are of different matches (a repeated one
leaves a null space of two dimensions, any vector of which is a solution).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from . import gpu_util as U  # noqa: E402
from .test_gpu_pnp import K, _gpu  # noqa: E402
from .test_oracle_tracking_pins import _problem  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hyps,iters,rounds", [(6, 1, 10, 2), (255, 63, 10, 2), (256, 64, 1, 1), (257, 65, 10, 3),
                                                 (65536, 8, 3, 2), (65537, 9, 3, 2), (500, 33, 0, 2), (500, 33, 10, 0)])
def test_pnp_at_edges(n, hyps, iters, rounds):
    from oracle import tracking as TK
    U.log(f"[gpu] pnp sizes n {n} hypotheses {hyps} iterations {iters} rounds {rounds}")
    small = n == 6
    X, uv, _, _, _ = _problem(n, 100 + hyps, outliers=0.0 if small else 0.2, noise=0.0 if small else 0.5)
    rng = np.random.default_rng(n)
    samples = np.stack([rng.permutation(n)[:6] for _ in range(hyps)])
    X32, uv32 = X.astype(np.float32).astype(np.float64), uv.astype(np.float32).astype(np.float64)
    ref = TK.pnp_ransac(X32, uv32, K, samples, thr=3.0, iters=iters, rounds=rounds)
    T, cnt, mask, scores, _ = _gpu(X, uv, samples, 3.0, iters=iters, rounds=rounds)
    good = ref["gaps"] > 1e-6
    assert (scores == ref["scores"])[good].mean() >= 0.98
    assert int(np.argmax(scores)) == ref["best"]
    np.testing.assert_allclose(T, ref["T"], atol=1e-9)
    if ref["margin"] > 1e-9:
        assert np.array_equal(mask, ref["inliers"]) and cnt == int(ref["inliers"].sum())
