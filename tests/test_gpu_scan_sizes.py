"""The offset scan's two forms and the emission in one or two launches agree: the same Gaussians
padded to record counts on either side of 2^20 (where both change) give the same bits, with
live counts at the edges of the scan's blocks (2048 records) and of a look-back window (64
blocks)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("live", [1, 7, 8, 9, 2047, 2048, 2049, 64 * 2048 + 1, 140_000])
def test_scan_forms_agree(live):
    U.log(f"[gpu] scan forms, {live} live records")
    sc = scenes.make_scene("c0", n=live, seed=live % 997)
    sc.log_scales -= 1.0 if live > 4096 else 0.0
    sc.log_scales[:, ::50] += 2.5
    params, T = U.to_dev(sc, torch)
    got = []
    for n in ((1 << 20), (1 << 20) + 1):
        pad = [p[..., :1].expand(*p.shape[:-1], n - live) for p in params]
        full = [torch.cat([p, q], -1).contiguous() for p, q in zip(params, pad)]
        full[0][2, live:] = -1e6  # behind the camera
        rast = Rasterizer(Window(sc.cams, T), n, binding.RasterConfig(pointmap_frame=1, tile=8), max_pairs=1 << 22)
        out, fs = rast.forward(full)
        got.append({k: v.cpu().numpy() for k, v in out.items()})
    assert all(np.array_equal(got[0][k], got[1][k]) for k in got[0])
