"""The float32 sums of the backward keep their order: gradients of one-wave views, bit for bit.

At one pixel per lane a wave sums each record's values over its 8 x 8 pixels in float32, as one
chain of fused multiply-adds in pixel order.  The parameter pass multiplies these sums by the conic
twice, so for near-degenerate Gaussians their last bits decide the leading digits of the gradients:
sums in another order are no less exact, and still move the norm of a window's gradients by more
than two runs of one form differ.  In a view of 8 x 8 pixels one wave adds each record once, so
nothing depends on the order of atomics and the gradients have to equal the stored ones.

``golden/one_wave_gradients.npz`` holds the gradients of the matrix-core form that first defined
the order (16x16x4 products over workgroups); ``python -m tests.test_gpu_one_wave_gradients PATH``
writes such a file.
"""
import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "one_wave_gradients.npz")
# Entries of one batch, of several and of several 64-entry steps; tiles of 1, 4 and 16 waves.
CASES = [(n, tile, frame, pose_only) for n in (1, 16, 19, 90)
         for tile, frame, pose_only in ((16, 1, False), (8, 0, False), (32, 2, False), (16, 1, True), (8, 0, True),
                                        (16, 2, True))]


def gradients(n, tile, frame, pose_only):
    rng = np.random.default_rng([n, tile, frame])
    f32 = lambda *a: torch.from_numpy(np.ascontiguousarray(np.concatenate(a), dtype=np.float32)).cuda()  # noqa: E731
    z = rng.uniform(1.0, 6.0, n)
    means = np.stack([rng.uniform(-0.5, 0.5, n) * z, rng.uniform(-0.5, 0.5, n) * z, z])
    log_scales = rng.uniform(-2.5, 0.0, (3, n))
    log_scales[0, ::3] = rng.uniform(-9.0, -6.0, n)[::3]  # flat: every third
    log_scales[1, ::6] = rng.uniform(-9.0, -6.0, n)[::6]  # and needles among them
    log_scales[2, ::6] += 1.5
    opacity = rng.normal(-1.0, 1.5, n)
    opacity[::7] = 9.0  # alpha is clamped, pixels stop
    params = (f32(means), f32(log_scales), f32(rng.normal(size=(4, n))), f32(opacity), f32(rng.uniform(0, 1, (3, n))))
    cam = Camera(width=8, height=8, fx=8.0, fy=8.0, cx=4.0, cy=4.0)
    T = f32(np.float32([1, 0, 0, 0.02, 0, 1, 0, -0.03, 0, 0, 1, 0.1])[None])
    up = {k: f32(rng.normal(size=c * 64)) for k, c in (("rgb", 3), ("depth", 1), ("alpha", 1), ("pointmap", 3))}
    for k, c in (("rgb", 3), ("depth", 1), ("alpha", 1), ("pointmap", 3)):
        up[k].view(c, 64)[:, 11:20] = 0.0  # pixels without a gradient
    rast = Rasterizer(Window([cam], T), n, binding.RasterConfig(pointmap_frame=frame, tile=tile, bg=(0.1, 0.2, 0.3)),
                      max_pairs=1 << 16)
    out, fs = rast.forward(params)
    pose = torch.zeros(1, 6, device="cuda")
    if pose_only:
        rast.pose_backward_into(params, out, up, fs, pose)
        return {"pose": pose.cpu().numpy()}
    grads = rast.zero_grads(params)
    rast.backward_into(params, out, up, fs, grads, pose)
    return {"pose": pose.cpu().numpy(), **{k: g.cpu().numpy() for k, g in grads.items()}}


def key(n, tile, frame, pose_only, name):
    return f"{n}_{tile}_{frame}_{int(pose_only)}_{name}"


@pytest.mark.parametrize("n,tile,frame,pose_only", CASES)
def test_one_wave_gradients_keep_their_bits(n, tile, frame, pose_only):
    U.log(f"[gpu] one-wave gradients n {n} tile {tile} frame {frame} pose only {pose_only}")
    golden = np.load(GOLDEN)
    for name, got in gradients(n, tile, frame, pose_only).items():
        want = golden[key(n, tile, frame, pose_only, name)]
        assert np.linalg.norm(want) > 0, name
        differ = int((got.view(np.uint32) != want.view(np.uint32)).sum())
        assert differ == 0, f"{name}: {differ} of {want.size} differ, at most by {np.abs(got - want).max()}"


if __name__ == "__main__":
    np.savez_compressed(sys.argv[1], **{key(*c, name): g for c in CASES for name, g in gradients(*c).items()})
    print("wrote", sys.argv[1], flush=True)
