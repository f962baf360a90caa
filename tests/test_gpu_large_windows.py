"""Windows above 65536 waves: the workgroup forward that does not count, and the backward there.

At one pixel per lane a larger window is composited by workgroups, a smaller one by independent
waves.  One view of 2304x2048 pixels has 73728 waves.  Its images and marks have to equal those of
the counting forward (another instantiation), and inside a crop with the same origin those of a
view of the crop's size, which the independent waves render: the same fragments in the same
order, bit for bit.  Its gradients are compared with the reduce-scatter form's under the bounds
of the gradient tests: the sums run over thousands of waves, in the order of the atomics.
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

W, H, CW, CH = 2304, 2048, 1024, 736
N = 4000


def inputs(seed):
    rng = np.random.default_rng(seed)
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    z = rng.uniform(2.0, 6.0, N)
    z[::50] = -1.0  # behind the camera: not marked
    x, y = (rng.uniform(0, W, N) - 500) / 1500 * z, (rng.uniform(0, H, N) - 400) / 1500 * z
    opacity = rng.normal(0.0, 1.5, N)
    opacity[::5] = 9.0
    return (f32(np.stack([x, y, z])), f32(rng.uniform(-4.5, -1.5, (3, N))), f32(rng.normal(size=(4, N))), f32(opacity),
            f32(rng.uniform(0, 1, (3, N))))


def render(params, width, height, **kw):
    # Without the Jacobian's clamp the records do not depend on the view's size.
    cfg = binding.RasterConfig(mark_visible=1, jac_clamp=1e6, bg=(0.1, 0.2, 0.3), **kw)
    T = torch.tensor([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]], dtype=torch.float32, device="cuda")
    rast = Rasterizer(Window([Camera(width, height, 1500.0, 1500.0, 500.0, 400.0)], T), N, cfg)
    out, fs = rast.forward(params)
    lay = U.frame_layout(rast.win.n_tiles(cfg.tile), rast.win.n_pixels, N)
    marks = fs[lay["visible"]:lay["visible"] + N].cpu().numpy() != 0
    images = {k: v.view(-1, height, width) for k, v in out.items()}
    return rast, out, fs, images, marks


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("frame", [0, 1, 2])
def test_forward_and_backward_of_a_large_view(tile, frame):
    U.log(f"[gpu] large view {W}x{H} tile {tile} frame {frame}")
    assert W * H // 64 > 65536 > CW * CH // 64
    params = inputs(10 * tile + frame)
    rast, out, fs, images, marks = render(params, W, H, tile=tile, pointmap_frame=frame)
    counted = render(params, W, H, tile=tile, pointmap_frame=frame, count_work=1)
    crop = render(params, CW, CH, tile=tile, pointmap_frame=frame)
    assert 0 < marks.sum() < N and np.array_equal(marks, counted[4]) and not (crop[4] & ~marks).any()
    for k, got in images.items():
        assert torch.equal(got, counted[3][k]), k
        assert torch.equal(got[:, :CH, :CW], crop[3][k]), k
    rng = np.random.default_rng(tile)
    up = {k: torch.from_numpy(rng.normal(size=v.numel()).astype(np.float32)).cuda() for k, v in out.items()}
    got = []
    for lane_reduce in (0, 1):
        rast.cfg = dataclasses.replace(rast.cfg, bwd_lane_reduce=lane_reduce)
        grads, pose = rast.zero_grads(params), torch.zeros(1, 6, device="cuda")
        rast.backward_into(params, out, up, fs, grads, pose)
        alone = torch.zeros(1, 6, device="cuda")
        rast.pose_backward_into(params, out, up, fs, alone)
        got.append({**grads, "pose": pose, "pose alone": alone})
    for k, want in got[1].items():
        U.check_grad(k, got[0][k].cpu().numpy(), want.cpu().numpy())
