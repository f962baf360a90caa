"""A Gaussian with a colour that is not finite spoils the pixels of the waves that take it, no others.

The workgroup forms leave out an entry that no pixel of a wave accepts.  The forms by independent
waves composite such entries with weight 0, which adds nothing, unless a colour (or an upstream
gradient) is not finite: 0 times infinity is NaN.  The images of the two forward forms have to be
equal bit for bit, NaN included, and the two backward forms have to spoil the gradients of the
same Gaussians.  Elsewhere they agree as float32 sums do: some 100 additions and tenfold
cancellation, 100 * 10 * 2^-24 = 6e-5 of the largest value.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding, scenes  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


def render(sc, **kw):
    params, T = U.to_dev(sc, torch)
    rast = Rasterizer(Window(sc.cams, T), sc.n, binding.RasterConfig(bg=(0.1, 0.2, 0.3), **kw), max_pairs=1 << 18)
    out, fs = rast.forward(params)
    return rast, params, out, fs


def scene(n, seed, bad):
    sc = scenes.make_scene("c0", n=n, seed=seed)
    sc.cams[0] = dataclasses.replace(sc.cams[0], width=93, height=61, cx=46.5, cy=30.5)
    sc.opacity_logit[::3] += 9.0
    sc.log_scales -= 0.5
    rast, params, out, fs = render(sc)
    grads = rast.zero_grads(params)
    rast.backward_into(params, out, {"rgb": torch.ones_like(out["rgb"])}, fs, grads)
    seen = np.argsort(-grads["rgb"][0].cpu().numpy())  # most visible first
    for k, value in enumerate(bad):
        sc.rgb[k % 3, seen[k + 1]] = value
    return sc


@pytest.mark.parametrize("tile,frame", [(16, 1), (8, 0), (32, 2)])
@pytest.mark.parametrize("n,bad", [(40, [np.inf]), (400, [np.nan]), (401, [np.inf, -np.inf, np.nan]), (400, [])])
def test_images(n, bad, tile, frame):
    U.log(f"[gpu] non-finite colours n {n} {bad} tile {tile} frame {frame}")
    sc = scene(n, n + tile, bad)
    waves, groups = (render(sc, tile=tile, pointmap_frame=frame, count_work=c)[2] for c in (0, 1))
    for k in waves:
        a, b = waves[k].cpu().numpy(), groups[k].cpu().numpy()
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32)) or \
            (np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[~np.isnan(a)], b[~np.isnan(b)])), k
    if bad:
        spoilt = ~np.isfinite(waves["rgb"].cpu().numpy())
        assert 0 < spoilt.sum() < spoilt.size


@pytest.mark.parametrize("tile,ppl,frame", [(16, 1, 1), (16, 2, 0), (8, 1, 2), (32, 4, 1)])
@pytest.mark.parametrize("n,bad,bad_up", [(40, [np.inf], 0), (400, [np.nan], 0), (401, [np.inf, -np.inf, np.nan], 0),
                                          (400, [], 1), (400, [np.inf], 2), (400, [], 0)])
def test_gradients(n, bad, bad_up, tile, ppl, frame):
    """ppl: of the forward (with others than 1 the backward tests every entry of the list)."""
    U.log(f"[gpu] non-finite gradients n {n} {bad} upstream {bad_up} tile {tile} ppl {ppl} frame {frame}")
    sc = scene(n, n + tile, bad)
    rast, params, out, fs = render(sc, tile=tile, pixels_per_lane=ppl, pointmap_frame=frame)
    up = {k: torch.from_numpy(v.reshape(-1)).cuda() for k, v in scenes.upstream_grads(sc, seed=n)[0].items()}
    for v in up.values():  # the right half has no upstream gradient
        v.view(-1, 61, 93)[:, :, 50:] = 0.0
    for k in range(bad_up):
        up["rgb"].view(3, 61, 93)[k, 20 + k, 10 + 9 * k] = np.nan
    got = []
    for lane_reduce in (0, 1):
        rast.cfg = dataclasses.replace(rast.cfg, pixels_per_lane=1, bwd_lane_reduce=lane_reduce)
        grads, pose = rast.zero_grads(params), torch.zeros(1, 6, device="cuda")
        rast.backward_into(params, out, up, fs, grads, pose)
        got.append({**{k: g.cpu().numpy() for k, g in grads.items()}, "pose": pose.cpu().numpy()})
    # A Gaussian is spoilt if any of its gradients is (the forms differ in which of them).
    params = ("means", "log_scales", "quats", "opacity_logit", "rgb")
    fine = [np.all([np.isfinite(g[k].reshape(-1, n)).all(axis=0) for k in params], axis=0) for g in got]
    assert np.array_equal(fine[0], fine[1]), f"spoilt: {np.sum(~fine[0])}, {np.sum(~fine[1])}"
    assert np.array_equal(np.isfinite(got[0]["pose"]), np.isfinite(got[1]["pose"]))
    for k in params if fine[0].any() else ():
        a, want = (g[k].reshape(-1, n)[:, fine[0]] for g in got)
        assert np.all(np.abs(a - want) <= 6e-5 * np.abs(want).max()), k
    if bad or bad_up:
        assert 0 < fine[0].sum() < n
