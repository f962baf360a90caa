"""The radix sort's forms give the same lists.

Sorts take 4, 8 or 16 ranking steps per tile by their capacity (up to 2^19, up to 2^21 and more),
the first two with digit totals by atomics and look-back in the first pass.  The same Gaussians,
rendered with pair capacities and padded to record counts on either side of both limits, have to
give the same bits: the sort is stable and exact whatever its form.  Key counts run over the
edges of the tiles (2048 and 4096 keys).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu

LIMITS = (1 << 19, 1 << 21)


def _render(sc, params, T, n, pairs, db):
    if n > params[0].shape[-1]:  # Gaussians behind the camera: no tile pairs
        pad = [p[..., :1].expand(*p.shape[:-1], n - p.shape[-1]) for p in params]
        params = [torch.cat([p, q], -1).contiguous() for p, q in zip(params, pad)]
        params[0][2, -pad[0].shape[-1]:] = -1e6
    rast = Rasterizer(Window(sc.cams, T), n, binding.RasterConfig(pointmap_frame=1, sort_digit_bits=db), max_pairs=pairs)
    out, fs = rast.forward(params)
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("db", [8, 5])
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4095, 4097, 9000])
def test_sort_forms_agree(n, db):
    U.log(f"[gpu] sort forms n {n} digit bits {db}")
    sc = scenes.make_scene("c0", n=n, seed=n)
    params, T = U.to_dev(sc, torch)
    want = _render(sc, params, T, n, 1 << 18, db)
    for pairs in [x + d for x in LIMITS for d in (0, 1)]:
        got = _render(sc, params, T, n, pairs, db)
        assert all(np.array_equal(got[k], want[k]) for k in want), pairs


@pytest.mark.parametrize("records", [x + d for x in LIMITS for d in (0, 1)])
def test_record_counts_agree(records):
    U.log(f"[gpu] sort forms with {records} records")
    sc = scenes.make_scene("c0", n=6000, seed=5)
    params, T = U.to_dev(sc, torch)
    want = _render(sc, params, T, 6000, 1 << 18, 8)
    got = _render(sc, params, T, records, 1 << 18, 8)
    assert all(np.array_equal(got[k], want[k]) for k in want)
