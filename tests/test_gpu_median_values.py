"""Median depth of images whose values crowd in few bins or spread over many.

The selection's histograms take one atomic for each of the first bins that a wave meets and single
ones for the rest.  Images of one depth (every lane in one bin), of few, of depths over 17 decades
(every lane in another top bin), with and without pixels that count for nothing; the median is
exact.  Neither kind may take much longer than ordinary depths: at 16 views of 1920x1080 one depth
took 1.2 times and 17 decades 2.7 times as long, and both take 0.9 times now.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402
from .test_gpu_shared_scratch import lower_median  # noqa: E402

pytestmark = pytest.mark.gpu


def depths(kind, n, seed=1):
    g = torch.Generator("cuda").manual_seed(seed)
    u = torch.rand(n, device="cuda", generator=g)
    return {"ordinary": 0.5 + 5.0 * u, "one": torch.full_like(u, 2.5), "few": torch.round(1 + 4 * u) / 4,
            "decades": torch.exp(40.0 * u - 20.0), "two": torch.where(u < 0.5, 1.0, 1.0 + 2.0 ** -23)}[kind]


def window(width, height, views):
    T = torch.zeros(views, 12, device="cuda")
    T[:, [0, 5, 10]] = 1.0
    return Rasterizer(Window([Camera(width, height, 500.0, 500.0, width / 2, height / 2)] * views, T), 1)


@pytest.mark.parametrize("kind", ["ordinary", "one", "few", "decades", "two"])
@pytest.mark.parametrize("width,height,views,empty", [(1, 1, 1, 0.0), (63, 1, 2, 0.0), (65, 3, 3, 0.3), (160, 120, 2, 0.9),
                                                      (317, 237, 4, 0.5)])
def test_median(kind, width, height, views, empty):
    U.log(f"[gpu] median {kind} {views} x {width}x{height} empty {empty}")
    rast = window(width, height, views)
    n = rast.win.n_pixels
    d = depths(kind, n, seed=width)
    out = torch.rand(n, device="cuda", generator=torch.Generator("cuda").manual_seed(views)) < empty
    d[out] = torch.where(torch.arange(n, device="cuda") % 2 == 0, 0.0, -1.0)[out]
    got = rast.median_depth(d).cpu().numpy()
    h = d.cpu().numpy().reshape(views, -1)
    assert np.array_equal(got, np.float32([lower_median(x) for x in h]))


def test_time_does_not_depend_on_the_values():
    U.log("[gpu] median times")
    rast = window(1920, 1080, 16)
    t = {}
    for kind in ("ordinary", "one", "decades"):
        d, runs = depths(kind, rast.win.n_pixels), []
        for _ in range(9):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                rast.median_depth(d)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b) * 200)
        t[kind] = float(np.median(runs))
    U.log(f"  us: {t}")
    assert t["one"] <= 1.1 * t["ordinary"] and t["decades"] <= 1.5 * t["ordinary"], t
