"""The sort's forms at the edges of their tiles: every form gives the same frame, bit for bit.

A sort takes 4, 8 or 16 ranking steps by its capacity (2^19 and 2^21), so that its tiles hold 2048,
4096 or 8192 keys.  Gaussians of one tile each make the number of pairs equal to their own, so both
sorts have n keys: n at the edges of each tile size, every form of the pair sort (by the frame
state's capacity) with every form of the depth sort (by records behind the camera that pad the
window).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu

W, H, TILE = 640, 480, 16


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 16385])
@pytest.mark.parametrize("bits", [8, 5])
def test_sort_forms_at_tile_edges(n, bits):
    U.log(f"[gpu] sort edges n {n} digit bits {bits}")
    rng = np.random.default_rng([n, bits])
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    # At a pixel inside a tile, with a footprint of two or three pixels.
    i, j = rng.integers(0, W // TILE, n) * TILE + 7, rng.integers(0, H // TILE, n) * TILE + 8
    z = rng.choice(np.linspace(1.0, 5.0, 997), n)  # equal depths too: ties keep the records' order
    params = [f32(np.stack([(i - 320) / 500 * z, (j - 240) / 500 * z, z])), f32(np.full((3, n), -7.0)),
              f32(rng.normal(size=(4, n))), f32(rng.uniform(-3, 0, n)), f32(rng.uniform(0, 1, (3, n)))]
    T = f32([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]])
    win = Window([Camera(W, H, 500.0, 500.0, 320.0, 240.0)], T)
    first = None
    for records in (n, (1 << 19) + 1, (1 << 21) + 1):
        pad = [p[..., :1].expand(*p.shape[:-1], records - n) for p in params]
        full = [torch.cat([p, q], -1).contiguous() for p, q in zip(params, pad)]
        full[0][2, n:] = -1.0
        for pairs in (1 << 19, 1 << 21, (1 << 21) + 1):
            rast = Rasterizer(win, records, binding.RasterConfig(tile=TILE, sort_digit_bits=bits), max_pairs=pairs)
            out, _ = rast.forward(full)
            assert rast.pairs == n and rast.max_pairs == pairs
            if first is None:
                first = out
                assert float(out["alpha"].max()) > 0
            assert all(torch.equal(out[k], first[k]) for k in out), (records, pairs)
