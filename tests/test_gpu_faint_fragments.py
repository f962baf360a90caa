"""Fragments too faint to change the transmittance keep their gradients.

With a small alpha_min a fragment may have an alpha below 2^-25: T (1 - alpha) rounds to T, but the
fragment contributes alpha T to the images, so the backward has to walk it.  The forward by
independent waves bounds the backward's walk per pixel; the counting forward (workgroups) notes
the last contributing entry itself.  From either the backward walks the same fragments, and in a
view of one wave it adds them in one order: equal gradients, bit for bit.  The faint Gaussians'
colour gradients are sums of alpha times the upstream gradient, all of one sign here: not zero.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130])
@pytest.mark.parametrize("tile,frame,behind,opaque", [(16, 1, 0, 0), (8, 0, 3, 0), (32, 2, 1, 0), (16, 1, 100, 4),
                                                      (8, 2, 100, 4)])
def test_faint_fragments_have_gradients(n, tile, frame, behind, opaque):
    """n faint Gaussians, then opaque ones that stop some of the pixels, then visible ones (or, behind
    opaque ones, faint ones again)."""
    U.log(f"[gpu] faint fragments n {n} tile {tile} frame {frame} opaque {opaque} behind {behind}")
    rng = np.random.default_rng([n, tile])
    m = n + opaque + behind
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    z = np.sort(rng.uniform(2.0, 3.0, m))
    log_scales = np.full((3, m), 1.0)
    log_scales[:, n:n + opaque] = -0.7  # 1.6 pixels
    opacity = np.full(m, -18.0)  # sigmoid 1.5e-8 < 2^-25
    opacity[n:n + opaque] = 9.0
    if not opaque:
        opacity[n:] = 0.5
    params = (f32(np.stack([rng.uniform(-0.3, 0.3, m), rng.uniform(-0.3, 0.3, m), z])), f32(log_scales),
              f32(rng.normal(size=(4, m))), f32(opacity), f32(rng.uniform(0.2, 1, (3, m))))
    T = f32(np.float32([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]]))
    up = {k: f32(rng.uniform(0.5, 1.5, c * 64)) for k, c in (("rgb", 3), ("depth", 1), ("pointmap", 3))}
    got = []
    for count in (1, 0):
        cfg = binding.RasterConfig(pointmap_frame=frame, tile=tile, alpha_min=1e-10, count_work=count)
        rast = Rasterizer(Window([Camera(8, 8, 8.0, 8.0, 4.0, 4.0)], T), m, cfg, max_pairs=1 << 16)
        out, fs = rast.forward(params)
        grads, pose = rast.zero_grads(params), torch.zeros(1, 6, device="cuda")
        rast.backward_into(params, out, up, fs, grads, pose)
        got.append({**{k: g.cpu().numpy() for k, g in grads.items()}, "pose": pose.cpu().numpy()})
    assert np.all(got[0]["rgb"] > 0)
    if opaque:
        T_final = 1.0 - out["alpha"].cpu().numpy()
        assert (T_final < 2e-2).any() and (T_final > 0.5).any()
    for k, want in got[0].items():
        assert np.array_equal(got[1][k], want), k
