"""The large window (16 views of 1920x1080, 3M Gaussians) at one pixel per lane, against the oracle.

Its 522k waves take the workgroup forward and the backward by independent waves.  The tile edges are
the autotuner's usual choices; inputs, checks and bounds are those of the full-size tests.
"""
import pytest

from . import test_gpu_fullsize as full
from .test_gpu_fullsize import lib  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [32, 16])
def test_large_window_at_one_pixel_per_lane(lib, oracle, tile):  # noqa: F811
    full.test_full_window(lib, oracle, "c4", tile, 1, None, 8)
