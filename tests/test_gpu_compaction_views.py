"""The compaction over several views, each with its own size and pose, against single views.

A segment of live bits and a large record belong to one view: taken for another's, they would get
its footprint.  Every view of a window has to come out bit for bit as it does alone, and the
window's pairs have to be the sum of the views'.  Gaussian counts lie around the 64 of a segment
(so that views begin inside a word's range), and beyond the 8192 segments from which the live bits
are added up in a launch of their own.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window, split_views  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu

CAMS = [Camera(333, 211, 300.0, 300.0, 160.0, 100.0), Camera(96, 160, 90.0, 95.0, 48.0, 80.0),
        Camera(401, 97, 350.0, 300.0, 200.0, 50.0), Camera(64, 64, 60.0, 60.0, 30.0, 33.0)]


def pose(k):
    a = 0.15 * k
    return [np.cos(a), 0, np.sin(a), 0.1 * k, 0, 1, 0, -0.05 * k, -np.sin(a), 0, np.cos(a), 0.2 * k]


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 5000, 180_001])
@pytest.mark.parametrize("tile", [8, 16])
def test_views_of_a_window_come_out_as_alone(n, tile):
    U.log(f"[gpu] compaction over views n {n} tile {tile}")
    rng = np.random.default_rng([n, tile])
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    z = rng.uniform(-1.0, 6.0, n)  # some behind the cameras
    z[0] = 3.0
    log_scales = rng.uniform(-5.0, -3.0, (3, n))
    every = max(1, min(40, n // 3))
    log_scales[:, ::every] = rng.uniform(0.0, 1.0, (3, n))[:, ::every]  # large ones in every view
    means = np.stack([rng.uniform(-2, 2, n), rng.uniform(-1, 1, n), z])
    means[:2, 0] = 0.0
    params = (f32(means), f32(log_scales), f32(rng.normal(size=(4, n))), f32(rng.normal(-1, 1, n)),
              f32(rng.uniform(0, 1, (3, n))))
    T = f32([pose(k) for k in range(len(CAMS))])
    cfg = binding.RasterConfig(tile=tile, bg=(0.1, 0.2, 0.3))
    window = Window(CAMS, T)
    rast = Rasterizer(window, n, cfg)
    out, _ = rast.forward(params)
    pairs = 0
    for v, cam in enumerate(CAMS):
        one = Rasterizer(Window([cam], T[v:v + 1].contiguous()), n, cfg)
        want, _ = one.forward(params)
        pairs += one.pairs
        for k, c in (("rgb", 3), ("depth", 1), ("alpha", 1), ("pointmap", 3)):
            assert torch.equal(split_views(window, out[k], c)[v].reshape(-1), want[k]), (v, k)
    assert rast.pairs == pairs
    # The first Gaussian alone has more than the 64 pairs of an ordinary record in the largest view.
    alone = Rasterizer(Window(CAMS[:1], T[:1].contiguous()), 1, cfg)
    alone.forward([p[..., :1].contiguous() for p in params])
    assert alone.pairs > 64
