"""The backward's two ways of forming the per-record sums agree.

With one pixel per lane, independent waves walk four entries at a time, stage them 16 at a time
and add their sums eight at a time; settings.bwd_lane_reduce selects the workgroup form, which
takes one entry at a time and adds lane by lane.  The list lengths run over the edges of these
groups and of the 64-entry steps of the bit planes; opaque Gaussians clamp alpha and stop pixels.

Both add the same fragments in float32: a sum over up to 64 pixels, then atomics over a few waves
and the later chain to the parameters.  An addition rounds to 2^-24 of the running sum, so some
100 of them and tenfold cancellation leave 100 * 10 * 2^-24 = 6e-5 of the largest value.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 63, 64, 65, 80, 81, 700])
@pytest.mark.parametrize("tile,frame,pose_only", [(16, 1, False), (16, 1, True), (8, 0, False), (32, 2, False),
                                                  (16, 0, True), (16, 2, True)])
def test_independent_waves_equal_lane_sums(n, tile, frame, pose_only):
    width, height = (45, 37) if n % 2 else (16, 16)
    U.log(f"[gpu] backward forms n {n} tile {tile} frame {frame} pose only {pose_only} view {width}x{height}")
    sc = scenes.make_scene("c0", n=n, seed=3 * n + width)
    sc.cams[0] = dataclasses.replace(sc.cams[0], width=width, height=height, cx=width / 2, cy=height / 2)
    sc.opacity_logit[::3] += 9.0
    sc.log_scales += 1.0
    params, T = U.to_dev(sc, torch)
    up = {k: torch.from_numpy(v.reshape(-1)).cuda() for k, v in scenes.upstream_grads(sc, seed=n)[0].items()}
    rast = Rasterizer(Window(sc.cams, T), n, binding.RasterConfig(pointmap_frame=frame, tile=tile, bg=(0.1, 0.2, 0.3)),
                      max_pairs=1 << 16)
    out, fs = rast.forward(params)
    got = []
    for lane_reduce in (0, 1):
        rast.cfg.bwd_lane_reduce = lane_reduce
        grads = None if pose_only else rast.zero_grads(params)
        pose = torch.zeros(1, 6, device="cuda")
        rast.backward_into(params, out, up, fs, grads, pose)
        got.append({"pose": pose.cpu().numpy(), **({} if pose_only else {k: g.cpu().numpy() for k, g in grads.items()})})
    for k, want in got[1].items():
        assert np.all(np.isfinite(got[0][k])), k
        assert np.all(np.abs(got[0][k] - want) <= 6e-5 * np.abs(want).max()), k
