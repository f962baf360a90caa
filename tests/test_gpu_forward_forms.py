"""The two forms of the forward compositing kernel give the same images, marks and gradients.

Small windows are composited by independent waves, large ones and counting renders by
workgroups; both evaluate the same expressions per pixel in the same order, so their images
are equal bit for bit.  A counting render (settings.count_work) selects the workgroup form.
The list lengths run over the edges of the 64-entry chunks (0, 1, 63, 64, 65, 128, ...), with
opaque Gaussians that clamp alpha and stop pixels in the middle of a chunk.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


def _scene(n, width, height, opaque):
    sc = scenes.make_scene("c0", n=max(n, 1), seed=n + width)
    sc.cams[0] = dataclasses.replace(sc.cams[0], width=width, height=height, cx=width / 2, cy=height / 2)
    if opaque:
        sc.opacity_logit[::3] += 9.0
        sc.log_scales += 1.0
    return sc


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 128, 129, 700])
@pytest.mark.parametrize("tile,frame,opaque", [(16, 1, True), (8, 0, False), (32, 2, True)])
def test_independent_waves_equal_workgroups(n, tile, frame, opaque):
    width, height = (45, 37) if n % 2 else (16, 16)
    U.log(f"[gpu] forward forms n {n} tile {tile} frame {frame} view {width}x{height}")
    sc = _scene(n, width, height, opaque)
    params, T = U.to_dev(sc, torch)
    params = [p[..., :n].contiguous() for p in params]
    cfg = binding.RasterConfig(pointmap_frame=frame, tile=tile, mark_visible=1, bg=(0.1, 0.2, 0.3))
    up = {k: torch.from_numpy(v.reshape(-1)).cuda() for k, v in scenes.upstream_grads(sc, seed=n)[0].items()}
    got = []
    for count in (0, 1):
        rast = Rasterizer(Window(sc.cams, T), n, dataclasses.replace(cfg, count_work=count), max_pairs=1 << 16)
        out, fs = rast.forward(params)
        seen = rast.covisibility(fs)[2].cpu()
        grads = rast.zero_grads(params)
        pose = torch.zeros(1, 6, device="cuda")
        if n:
            rast.backward_into(params, out, up, fs, grads, pose)
        got.append(({k: v.cpu().numpy() for k, v in out.items()}, seen, {k: g.cpu().numpy() for k, g in grads.items()},
                    pose.cpu().numpy()))
    (img0, seen0, g0, p0), (img1, seen1, g1, p1) = got
    for k in img0:
        assert np.array_equal(img0[k], img1[k]), k
    assert torch.equal(seen0, seen1)
    # The same fragments, summed by atomics in another order: float rounding of the sums only.
    for k in g0:
        scale = np.abs(g1[k]).max() if g1[k].size else 0.0
        assert np.all(np.abs(g0[k] - g1[k]) <= 1e-4 * scale), k
    assert np.all(np.abs(p0 - p1) <= 1e-4 * np.abs(p1).max() + 1e-12)
