"""Median depth at the edges of its selection: values that share the top 11 or 22 bits, bins at
both ends of a round, one value, none, counts around a workgroup, negative values and zeros
(which do not count), against a sort: the lower median of the positive depths, exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding as B, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


def _bits(x):
    return np.asarray(x, dtype=np.uint32).view(np.float32)


@pytest.mark.parametrize("case", ["top", "low", "ends", "one", "none", "mixed"])
def test_median_at_edges(case):
    U.log(f"[gpu] median edges {case}")
    rng = np.random.default_rng(1)
    w, h = 37, 29
    n = w * h
    d = {"top": _bits(0x40000000 + rng.integers(0, 1 << 10, n)),            # equal in the first 22 bits
         "low": _bits(0x40000000 + (rng.integers(0, 1 << 11, n) << 10)),    # equal in the first 11
         "ends": _bits(rng.choice([1, 0x7f7fffff, 0x3fffffff, 0x40000000], n)),
         "one": np.where(np.arange(n) == 500, np.float32(3.5), np.float32(0)),
         "none": np.full(n, -1.0, np.float32),
         "mixed": np.where(rng.random(n) < 0.3, 0, rng.normal(2.0, 3.0, n)).astype(np.float32)}[case]
    sizes = [(w, h), (1, 1), (256, 1), (257, 1)]
    cams = [scenes.Camera(a, b, 50.0, 50.0, a / 2, b / 2) for a, b in sizes]
    views = [d] + [d[:a * b] for a, b in sizes[1:]]
    T = torch.zeros(len(cams), 12, device="cuda")
    T[:, 0] = T[:, 5] = T[:, 10] = 1.0
    rast = Rasterizer(Window(cams, T), 1, B.RasterConfig())
    got = rast.median_depth(torch.from_numpy(np.concatenate(views)).cuda()).cpu().numpy()
    for g, x in zip(got, views):
        pos = np.sort(x[x > 0])
        assert g == (pos[(pos.size - 1) // 2] if pos.size else np.float32(0)), case
