"""Scale alignment with patches taller than the 12 rows that a lane keeps: the rows beyond them are
read four at a time, so patch heights and image edges run over every remainder.

Against the float64 oracle under the bounds of the other alignment sizes; a mask of ones gives the
bits of no mask, and what the mask leaves out may be anything, NaN included.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding as B, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402
from .test_gpu_align_sizes import test_align_and_replace_at_edges as check_against_oracle  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("patch,width,height", [(13, 40, 26), (14, 50, 41), (15, 47, 46), (16, 64, 61), (17, 70, 50),
                                                (31, 64, 90), (64, 130, 77), (64, 64, 192)])
def test_tall_patches(patch, width, height):
    check_against_oracle(patch, width, height, 0)


@pytest.mark.parametrize("patch,width,height", [(13, 40, 26), (16, 64, 61), (64, 130, 77)])
def test_mask_of_tall_patches(patch, width, height):
    U.log(f"[gpu] align tall patch {patch} view {width}x{height}")
    cam = scenes.Camera(width, height, 60.0, 60.0, width / 2, height / 2)
    Xr = scenes.street_pointmap(cam, patch).astype(np.float32)
    Xp = scenes.noisy_prior(Xr, 0.9, patch + 1).astype(np.float32)
    T = torch.zeros(1, 12, device="cuda")
    T[:, 0] = T[:, 5] = T[:, 10] = 1.0
    rast = Rasterizer(Window([cam], T), 1, B.RasterConfig())

    def align(xr, xp, mask):
        res = rast.new_align_result()
        rast.align_scale_into(*(torch.from_numpy(x.reshape(-1)).cuda() for x in (xr, xp)), res,
                              None if mask is None else torch.from_numpy(mask.reshape(-1)).cuda(), B.AlignConfig(patch=patch))
        return res.cpu().numpy()
    ones = np.ones((height, width), np.float32)
    assert np.array_equal(align(Xr, Xp, None), align(Xr, Xp, ones))
    mask = (np.random.default_rng(patch).random((height, width)) > 0.4).astype(np.float32)
    spoilt_r, spoilt_p = Xr.reshape(3, height, width).copy(), Xp.reshape(3, height, width).copy()
    spoilt_r[:, mask == 0], spoilt_p[:, mask == 0] = np.nan, np.inf
    assert np.array_equal(align(Xr, Xp, mask), align(spoilt_r, spoilt_p, mask))
