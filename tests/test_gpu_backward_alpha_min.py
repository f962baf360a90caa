"""A backward with a larger alpha_min than its forward's leaves out the fragments below its own.

The settings of a backward are its caller's.  One broad Gaussian in front of one view: alpha is
known per pixel from the forward's alpha image, T = 1, so its colour gradient is the sum of
alpha times the upstream gradient over the pixels whose alpha reaches the backward's alpha_min.
Pixels within 1e-6 of it are given no upstream gradient.  64 to 3072 terms in float32, all of one
sign, each rounded to 2^-24 a few times, added in chains of at most 64: 1e-5 of the sum.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height", [(8, 8), (64, 48)])
@pytest.mark.parametrize("tile,ppl,frame,lane_reduce", [(16, 1, 1, 0), (8, 1, 0, 0), (32, 1, 2, 0), (16, 1, 1, 1), (16, 2, 1, 0)])
def test_backward_uses_its_own_alpha_min(width, height, tile, ppl, frame, lane_reduce):
    U.log(f"[gpu] backward alpha_min {width}x{height} tile {tile} ppl {ppl} frame {frame} lane reduce {lane_reduce}")
    f32 = lambda *a: torch.tensor(a, dtype=torch.float32, device="cuda")  # noqa: E731
    params = (f32([0.0], [0.0], [2.0]), f32([-1.5], [-1.2], [-1.0]), f32([1.0], [0.2], [-0.1], [0.3]), f32(1.0),
              f32([0.3], [0.6], [0.9]))
    T = f32([1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0])
    cfg = binding.RasterConfig(tile=tile, pixels_per_lane=ppl, pointmap_frame=frame, bwd_lane_reduce=lane_reduce)
    rast = Rasterizer(Window([Camera(width, height, float(width), float(width), width / 2, height / 2)], T), 1, cfg,
                      max_pairs=1 << 14)
    out, fs = rast.forward(params)
    alpha = out["alpha"].cpu().numpy().astype(np.float64)
    rng = np.random.default_rng(width + tile)
    g = rng.uniform(0.5, 1.5, (3, width * height)).astype(np.float32)
    for own in (1.0 / 255.0, 0.1, 0.3):
        g[:, np.abs(alpha - own) < 1e-6] = 0.0
        rast.cfg = dataclasses.replace(cfg, alpha_min=own)
        grads = rast.zero_grads(params)
        rast.backward_into(params, out, {"rgb": torch.from_numpy(g).cuda().reshape(-1)}, fs, grads)
        want = (alpha * (alpha >= own) * g).sum(axis=1)
        got = grads["rgb"].cpu().numpy().reshape(3)
        assert (alpha >= 0.3).any() and ((alpha > 0) & (alpha < 0.1)).any()
        assert np.all(np.abs(got - want) <= 1e-5 * want), (own, got, want)
