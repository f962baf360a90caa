"""Windows with more tile pairs than 32 bits count report an overflow and emit in bounds.

Screen-filling records in a view of 1920x1080 at 8 x 8 tiles have 32400 pairs each: 132560 of them
stay below 2^32, one more passes it.  The count has to be exact below and to stop at 2^32 - 1
from there on, in both forms of the offset scan (up to 2^20 records in one launch, more in two),
with ordinary records before, between and behind the large ones; a count that wrapped would pass
for a frame that fits.  Records behind the capacity emit nothing: the pairs within it are those
of the front records alone, so the images equal those of a window with the front records only
(at the same capacity, which they overflow as well).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu

CAM = Camera(1920, 1080, 1000.0, 1000.0, 960.0, 540.0)
TILES = 240 * 135
CAP = 100_000  # three large records and a part of the fourth


def gaussians(large, small):
    """large screen-filling ones from depth 4 on, small ones (a pair or a few) between 2 and 8."""
    n = large + small
    z = torch.empty(n, device="cuda")
    z[:large] = torch.linspace(4.0, 6.0, large, device="cuda", dtype=torch.float64).float()
    z[large:] = torch.linspace(2.0, 8.0, small, device="cuda", dtype=torch.float64).float() + 1e-3 if small else 0.0
    k = torch.arange(n, device="cuda", dtype=torch.float32)
    means = torch.stack([torch.sin(k) * 0.8, torch.cos(k) * 0.4, z])
    means[:2, :large] = 0.0
    log_scales = torch.full((3, n), -4.0, device="cuda")
    log_scales[:, :large] = 4.0
    quats = torch.zeros(4, n, device="cuda")
    quats[0] = 1.0
    opacity = torch.full((n,), -2.0, device="cuda")
    return means, log_scales, quats, opacity, torch.rand(3, n, device="cuda", generator=torch.Generator("cuda").manual_seed(n))


def forward(params, max_pairs=CAP):
    T = torch.tensor([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]], dtype=torch.float32, device="cuda")
    rast = Rasterizer(Window([CAM], T), params[0].shape[1], binding.RasterConfig(tile=8), max_pairs=max_pairs)
    out, fs = rast.forward(params, check=False)
    try:
        return out, binding.frame_status(fs, binding.stream_handle())
    except binding.CapacityError as e:
        return out, e.pairs


@pytest.mark.parametrize("large,small", [(132560, 0), (132561, 0), (132562, 3000), (265200, 0), (300, 1_100_000),
                                         (140_000, 1_000_000), (1_100_000, 2000)])
def test_pair_counts_saturate(large, small):
    U.log(f"[gpu] pair overflow, {large} large and {small} small records")
    params = gaussians(large, small)
    alone = forward([p[..., large:].contiguous() for p in params], max_pairs=1 << 24)[1] if small else 0
    out, pairs = forward(params)
    assert pairs == min(large * TILES + alone, 2 ** 32 - 1)
    # The front 3000 records in depth order hold more pairs than the capacity.
    order = torch.sort(params[0][2], stable=True).indices
    front = order[:torch.searchsorted(torch.cumsum((order < large).long(), 0), torch.tensor(5, device="cuda")) + 1]
    front = torch.sort(front).values  # the same order of records
    front_out, front_pairs = forward([p[..., front].contiguous() for p in params])
    assert front_pairs > CAP
    for k in out:
        assert torch.equal(out[k], front_out[k]), k


def test_forward_raises_beyond_any_capacity():
    U.log("[gpu] pair overflow, checked forward")
    params = gaussians(132561, 0)
    T = torch.tensor([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]], dtype=torch.float32, device="cuda")
    rast = Rasterizer(Window([CAM], T), params[0].shape[1], binding.RasterConfig(tile=8), max_pairs=CAP)
    with pytest.raises(binding.CapacityError):
        rast.forward(params)
