"""Pointmap replacement over windows of every size: the numbers of workgroups and the widths of its
accesses change with the window (4M and 12M pixels).

Eq. 14 in float64 from the same float32 inputs and scales, rounded once: equal but for the last bit,
where the compiler may contract a product and a sum; the count of replaced pixels is exact where no
pixel lies within 1e-9 of the limit.
"""
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding as B  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window, align_results  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height,views", [(3, 1, 1), (160, 120, 1), (161, 121, 3), (640, 480, 32), (1920, 1080, 2),
                                                (1920, 1080, 4), (1919, 1081, 4), (1920, 1080, 8), (4096, 3072, 1),
                                                (4097, 3073, 1)])
def test_replacement(width, height, views):
    U.log(f"[gpu] replacement {views} x {width}x{height}")
    T = torch.zeros(views, 12, device="cuda")
    T[:, [0, 5, 10]] = 1.0
    rast = Rasterizer(Window([Camera(width, height, 500.0, 500.0, width / 2, height / 2)] * views, T), 1)
    g = torch.Generator("cuda").manual_seed(width + views)
    P = rast.win.n_pixels
    Xr = torch.rand(3 * P, device="cuda", generator=g) + 1.0
    Xp = Xr * (1.0 + 0.6 * (torch.rand(3 * P, device="cuda", generator=g) - 0.5))
    res = rast.new_align_result()
    scales = 0.8 + 0.4 * torch.rand(views, device="cuda", generator=g, dtype=torch.float64)
    res.view(torch.float64).view(views, 3)[:, 0] = scales  # gspm_align_result: the scale first
    assert list(align_results(res)["scale"]) == list(scales.cpu().numpy())
    hat, count = torch.empty_like(Xr), torch.empty(views, dtype=torch.int32, device="cuda")
    rast.replace_pointmap_into(Xr, Xp, res, hat, count, eps_m=0.15)
    eps = float(torch.tensor(0.15, dtype=torch.float32))
    for v in range(views):
        a, b = 3 * rast.win.pix_off[v], 3 * rast.win.pix_off[v + 1]
        r, s = Xr[a:b].view(3, -1), scales[v] * Xp[a:b].view(3, -1).double()
        d, t = (r - s).norm(dim=0), eps * s.norm(dim=0)
        replaced = d > t
        clear = (d - t).abs() > 1e-9
        want = torch.where(replaced, s.float(), r)
        got = hat[a:b].view(3, -1)
        off = (got - want).abs() > (torch.nextafter(want.abs(), torch.full_like(want, 9e9)) - want.abs())
        assert not (off & clear).any(), v
        if clear.all():
            assert int(count[v]) == int(replaced.sum()), v
        assert int(count[v]) > 0 or width * height < 10
