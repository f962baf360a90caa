"""Compaction of the live records and large records (counted and emitted by groups of lanes) at
the edges of segments (64 Gaussians), tiles of segments and blocks, over several views.

The same Gaussians are rendered in another order: with distinct depths the lists, and so the
images, do not depend on it, but every record sits in another segment and lane.  Gaussians
near the camera cover more than 64 tiles; some lie behind it and leave gaps in the live bits.
The record counts include ones beyond half a million, which take one launch more.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


def _render(cams, T, params):
    n = params[0].shape[-1]
    rast = Rasterizer(Window(cams, T), n, binding.RasterConfig(pointmap_frame=1, tile=8, mark_visible=1), max_pairs=1 << 20)
    out, fs = rast.forward(params)
    return {k: v.cpu().numpy() for k, v in out.items()}, [x.cpu() for x in rast.covisibility(fs)]


@pytest.mark.parametrize("n,views", [(1, 1), (63, 2), (64, 3), (65, 3), (127, 1), (2047, 2), (2049, 2), (5000, 5),
                                     (1 << 19, 1), ((1 << 19) + 64, 1), (300_001, 2)])
def test_order_of_gaussians_does_not_matter(n, views):
    U.log(f"[gpu] compaction n {n} views {views}")
    live = min(n, 1500)
    sc = scenes.make_scene("c0", n=live, seed=n % 1000)
    sc.cams[0] = dataclasses.replace(sc.cams[0], width=200, height=150, cx=100.0, cy=75.0)
    params, T = U.to_dev(sc, torch)
    params[1][:, ::7] += 2.0  # large ones
    if n > live:  # the rest lies behind the camera
        pad = [p[..., :1].expand(*p.shape[:-1], n - live) for p in params]
        params = [torch.cat([p, q], -1).contiguous() for p, q in zip(params, pad)]
        params[0][2, live:] = -1e6
    cams, T = [sc.cams[0]] * views, T[:1].expand(views, -1).contiguous()
    want, covis = _render(cams, T, params)
    g = torch.Generator().manual_seed(n)
    order = torch.randperm(n, generator=g).cuda()
    got, covis2 = _render(cams, T, [p[..., order].contiguous() for p in params])
    z = params[0][2, :live]
    if torch.unique(z).numel() == live:  # ties keep record order, which differs
        assert all(np.array_equal(got[k], want[k]) for k in want)
        assert all(torch.equal(a, b) for a, b in zip(covis, covis2))
