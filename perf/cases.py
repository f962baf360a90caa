"""Performance cases: what a SLAM program asks of this library, through its public entry points.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same ranges, ``prepare(case,
seed)`` makes what a program holds before the call (inputs, the window, its Rasterizer and buffers),
``run(state)`` is one pass, ``work(case)`` the bytes and operations that pass cannot do without and
``exact(case, seed)`` the same results in float64 from plain torch.

Kinds of case:

* ``track``     one iteration of the tracking loop on one frame: render, window loss, pose gradient;
* ``map``       one mapping iteration over a window of keyframes: render, window loss, gradients of
                every Gaussian and pose, isotropic regulariser (``graph``: replayed from a capture);
* ``render``    one checked render, for evaluation or a new keyframe's pointmap;
* ``grad``      a program with a loss of its own: ``rasterize`` under autograd, dense upstream
                gradients on colour, depth, alpha and pointmap;
* ``keyframe``  the per-frame decision: render with marks, covisibility, median depth;
* ``pnp``       the pose of a new frame from 2D-3D matches (RANSAC + PnP);
* ``align``     scale alignment of a prior pointmap and its replacement, over a window.

Scenes are drawn on the GPU with the structure of ``scenes.py``: a street (ground plane and facades)
seen from keyframes along a trajectory, or Gaussians uniform on one small screen.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2507_03737_amd import binding as B
from paper_2507_03737_amd.render import MappingStep, Rasterizer, Window, rasterize
from paper_2507_03737_amd.scenes import Camera
from paper_2507_03737_amd.tracking import PnpConfig, pnp_ransac

DEV = "cuda"
NAMES = ("means", "log_scales", "quats", "opacity_logit", "rgb")
C3 = "960x640,960x640,960x640,1216x352,1216x352,1216x352,640x480,640x480"


def listed():
    return [
        # The smallest configuration: latency and launches of a tracking loop on a thumbnail.
        {"name": "track 160x120 2k", "kind": "track", "scene": "screen", "n": 2000, "sizes": "160x120"},
        # The tracking configuration: 500k Gaussians, one 960x640 frame.
        {"name": "track 960x640 500k", "kind": "track", "scene": "street", "n": 500_000, "sizes": "960x640"},
        # A low-resolution window early in a sequence, its iterations replayed from a captured graph.
        {"name": "map 3x 317x237 50k graph", "kind": "map", "scene": "street", "n": 50_000,
         "sizes": "317x237,317x237,317x237", "graph": True},
        # The mapping window of the benchmark: 1M Gaussians, 8 keyframes of uneven size.
        {"name": "map 8 views 1M", "kind": "map", "scene": "street", "n": 1_000_000, "sizes": C3},
        # The large window: 3M Gaussians, 16 keyframes of 1920x1080.
        {"name": "map 16x 1920x1080 3M", "kind": "map", "scene": "street", "n": 3_000_000,
         "sizes": ",".join(["1920x1080"] * 16)},
        # Rendering one frame (KITTI-like) for evaluation, with the overflow check.
        {"name": "render 1216x352 300k", "kind": "render", "scene": "street", "n": 300_000, "sizes": "1216x352"},
        # A loss of the caller's own under autograd, world-frame pointmap.
        {"name": "grad 1216x352 300k", "kind": "grad", "scene": "street", "n": 300_000, "sizes": "1216x352",
         "frame": 0},
        # Is this frame a keyframe?  The frame and the latest keyframe rendered with marks.
        {"name": "keyframe 2x 960x640 500k", "kind": "keyframe", "scene": "street", "n": 500_000,
         "sizes": "960x640,960x640"},
        # Pose initialisation from 20k matches, 20% of them wrong.
        {"name": "pnp 20000 1024", "kind": "pnp", "n": 20_000, "hypotheses": 1024},
        # Scale alignment and replacement of the window's priors.
        {"name": "align 8 views", "kind": "align", "sizes": C3, "patch": 10, "mask": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("track", "track", "map", "map", "map", "render", "grad", "keyframe", "pnp", "align"))
    if kind == "pnp":
        return {"kind": kind, "n": _log(rng, 200, 50_000), "hypotheses": _log(rng, 64, 2048)}
    views = {"track": 1, "render": rng.randint(1, 2), "grad": rng.randint(1, 3), "keyframe": rng.randint(2, 8)}.get(
        kind, rng.randint(1, 10))
    w = _log(rng, 120, 1300)
    size = "%dx%d" % (w, max(60, int(w * rng.uniform(0.3, 0.8))))
    case = {"kind": kind, "sizes": ",".join([size] * views)}
    if kind == "align":
        return dict(case, patch=rng.choice((7, 10, 10, 16)), mask=rng.random() < 0.5)
    case.update(scene="street", n=_log(rng, 5_000, 1_000_000))
    if kind == "grad":
        case["frame"] = rng.choice((0, 1, 2))
    if kind == "map" and rng.random() < 0.3:  # the other shape that the autotuner picks for windows
        case.update(tile=32, ppl=2)
    if kind == "map" and rng.random() < 0.3:
        case["graph"] = True
    return case


# ---- inputs ----------------------------------------------------------------------------------


def _cams(case):
    cams = []
    for s in case["sizes"].split(","):
        w, h = (int(x) for x in s.split("x"))
        cams.append(Camera(w, h, 128.0, 128.0, w / 2.0, h / 2.0) if case.get("scene") == "screen"
                    else Camera.fov80(w, h))
    return cams


def _uniform(g, lo, hi, *shape):
    return torch.rand(*shape, device=DEV, generator=g) * (hi - lo) + lo


def _street(g, n, tan_half):
    """Camera-frame centres: 70% on the ground 1.6 m below, 30% on facades beside the street."""
    z = torch.exp(_uniform(g, 0.0, math.log(80.0), n))
    ground = torch.rand(n, device=DEV, generator=g) < 0.7
    x = _uniform(g, -1.2, 1.2, n) * z * tan_half
    block = (z / 12.0).long()
    side = (torch.rand(n, device=DEV, generator=g) < 0.5).long()
    offset, height = _uniform(g, 4.0, 12.0, 2, 8), _uniform(g, 4.0, 15.0, 2, 8)
    front = torch.rand(n, device=DEV, generator=g) < 0.2
    xf = (2.0 * side - 1.0) * (offset[side, block] + front * _uniform(g, 0.0, 4.0, n))
    yf = 1.6 - torch.rand(n, device=DEV, generator=g) * height[side, block]
    zf = torch.where(front, 12.0 * block + 1.0, z)
    return torch.stack([torch.where(ground, x, xf), torch.where(ground, 1.6, yf), torch.where(ground, z, zf)])


def _scene(case, cams, g):
    """Gaussian parameters [rows][n] and poses T_cw [V][12] (float32, on the GPU)."""
    n, V = case["n"], len(cams)
    T = torch.zeros(V, 3, 4, device=DEV)
    if case["scene"] == "screen":
        c = cams[0]
        z = _uniform(g, 2.0, 20.0, n)
        u, v = _uniform(g, 0.0, c.width, n), _uniform(g, 0.0, c.height, n)
        means = torch.stack([(u - c.cx) * z / c.fx, (v - c.cy) * z / c.fy, z])
        T[:, :, :3] = torch.eye(3, device=DEV)
        scale, spread, logit, lspread = -2.5, 0.5, 0.0, 1.0
    else:
        yaw = _uniform(g, -math.radians(5.0), math.radians(5.0), V)
        R = torch.zeros(V, 3, 3, device=DEV)  # camera -> world
        R[:, 0, 0] = R[:, 2, 2] = torch.cos(yaw)
        R[:, 0, 2], R[:, 2, 0], R[:, 1, 1] = torch.sin(yaw), -torch.sin(yaw), 1.0
        C = torch.zeros(V, 3, device=DEV)
        C[:, 2] = 1.5 * torch.arange(V, device=DEV)
        local = _street(g, n, math.tan(math.radians(40.0)))
        owner = torch.randint(0, V, (n,), device=DEV, generator=g)
        means = (R[owner] * local.T[:, None, :]).sum(-1).T + C[owner].T
        T[:, :, :3] = R.transpose(1, 2)
        T[:, :, 3] = -(R.transpose(1, 2) * C[:, None, :]).sum(-1)
        scale, spread, logit, lspread = (-3.0, 0.7, 0.5, 1.5) if n <= 1_500_000 else (-3.5, 0.8, 0.5, 1.5)
    normal = lambda *s: torch.randn(*s, device=DEV, generator=g)  # noqa: E731
    q = normal(4, n)
    params = [means.contiguous(), scale + spread * normal(3, n), q / q.norm(dim=0), logit + lspread * normal(n),
              torch.rand(3, n, device=DEV, generator=g)]
    return params, T.reshape(V, 12).contiguous()


def _pointmap(cam, g):
    """Camera-frame pointmap [3][H][W] of a street: ground, two walls and a far backdrop."""
    jj, ii = torch.meshgrid(torch.arange(cam.height, device=DEV), torch.arange(cam.width, device=DEV), indexing="ij")
    rx, ry = (ii - cam.cx) / cam.fx, (jj - cam.cy) / cam.fy
    wall = _uniform(g, 6.0, 10.0, 2)
    z = torch.full_like(rx, 80.0)
    z = torch.where(ry > 1e-3, torch.minimum(z, 1.6 / ry.clamp(min=1e-3)), z)
    z = torch.minimum(z, torch.where(rx > 0, wall[0], wall[1]) / rx.abs().clamp(min=1e-3))
    z = z * (1.0 + 0.003 * torch.randn(z.shape, device=DEV, generator=g))
    return torch.stack([rx * z, ry * z, z])


def _prior(X, g, patch, wild):
    """The pointmap at another scale in every patch, with noise; with `wild`, a tenth of the patches at
    an unrelated scale and a hundredth of the pixels far off."""
    _, h, w = X.shape
    ph, pw = -(-h // patch), -(-w // patch)
    f = torch.full((ph, pw), 1.0 / 1.7, device=DEV) if wild else _uniform(g, 0.8, 1.25, ph, pw)
    if wild:
        bad = torch.rand(ph, pw, device=DEV, generator=g) < 0.1
        f = torch.where(bad, f * _uniform(g, 0.3, 3.0, ph, pw), f)
    s = f.repeat_interleave(patch, 0).repeat_interleave(patch, 1)[:h, :w]
    s = s * (1.0 + 0.01 * torch.randn(h, w, device=DEV, generator=g))
    if wild:
        far = torch.rand(h, w, device=DEV, generator=g) < 0.01
        s = torch.where(far, s * _uniform(g, 2.0, 5.0, h, w), s)
    return X * s


def _packed(planes):
    return torch.cat([p.reshape(-1) for p in planes]).contiguous()


def _inputs(case, seed):
    """Everything that is drawn: shared by prepare() and exact()."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    d = {}
    if case["kind"] == "pnp":
        n, H = case["n"], case["hypotheses"]
        d["cam"] = cam = Camera.fov80(960, 640)
        X = _pointmap(cam, g).reshape(3, -1)
        d["X"] = X[:, torch.randint(0, X.shape[1], (n,), device=DEV, generator=g)].contiguous()
        a = 0.05
        R = torch.tensor([[math.cos(a), 0, math.sin(a)], [0, 1, 0], [-math.sin(a), 0, math.cos(a)]], device=DEV)
        Y = (R[:, :, None] * d["X"][None]).sum(1) + torch.tensor([0.2, -0.05, 0.6], device=DEV)[:, None]
        uv = torch.stack([cam.fx * Y[0] / Y[2] + cam.cx, cam.fy * Y[1] / Y[2] + cam.cy])
        uv = uv + torch.randn(2, n, device=DEV, generator=g)
        bad = torch.rand(n, device=DEV, generator=g) < 0.2
        d["uv"] = (uv + bad * _uniform(g, 50.0, 150.0, 2, n)).contiguous()
        # Six different matches per hypothesis: one of each sixth of the list.
        d["samples"] = (torch.arange(6, device=DEV) * (n // 6)
                        + torch.randint(0, n // 6, (H, 6), device=DEV, generator=g)).int().contiguous()
        d["T_ak"] = torch.tensor([1, 0, 0, 0.3, 0, 1, 0, -0.1, 0, 0, 1, 2.0], device=DEV)
        return d
    d["cams"] = cams = _cams(case)
    P = sum(c.width * c.height for c in cams)
    if case["kind"] == "align":
        d["T"] = torch.zeros(len(cams), 12, device=DEV)
        Xr = [_pointmap(c, g) for c in cams]
        d["Xr"], d["Xp"] = _packed(Xr), _packed([_prior(x, g, case["patch"], True) for x in Xr])
        d["mask"] = (torch.rand(P, device=DEV, generator=g) < 0.9).float() if case["mask"] else None
        return d
    d["params"], d["T"] = _scene(case, cams, g)
    if case["kind"] in ("track", "map"):
        d["target"] = torch.rand(3 * P, device=DEV, generator=g)
        d["prior"] = _packed([_prior(_pointmap(c, g), g, 8, False) for c in cams])
    if case["kind"] == "grad":
        normal = lambda k: torch.randn(k * P, device=DEV, generator=g)  # noqa: E731
        d["up"] = {"rgb": normal(3), "depth": normal(1), "alpha": normal(1), "pointmap": normal(3)}
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "pnp":
        return dict(d, kind=kind, cfg=PnpConfig(n_hypotheses=case["hypotheses"], threshold=3.0), ctx=B.Context())
    win = Window(d["cams"], d["T"])
    s = dict(d, kind=kind, win=win)
    if kind == "align":
        rast = s["rast"] = Rasterizer(win, 1)
        s["cfg"] = B.AlignConfig(patch=case["patch"])
        s["result"], s["hat"] = rast.new_align_result(), torch.empty_like(d["Xr"])
        s["replaced"] = torch.empty(win.n_views, dtype=torch.int32, device=DEV)
        return s
    params = d["params"]
    cfg = B.RasterConfig(tile=case.get("tile", 16), pixels_per_lane=case.get("ppl", 1),
                         pointmap_frame=case.get("frame", 1), mark_visible=int(kind == "keyframe"))
    # One checked render finds the window's pair count; a program keeps a list of that size.
    probe = Rasterizer(win, case["n"], cfg)
    probe.forward(params)
    rast = s["rast"] = Rasterizer(win, case["n"], cfg, max_pairs=int(probe.pairs * 1.3) + 4096)
    del probe
    rast.reserve()
    if kind == "map":
        step = s["step"] = MappingStep(rast, params, d["target"], d["prior"])
        s["iso"] = torch.empty(1, device=DEV)
        if case.get("graph"):
            step.capture()
        return s
    if kind in ("track", "keyframe"):
        s["out"], s["fs"] = rast.new_outputs(), rast.new_frame_state()
    if kind == "track":
        s["scale"] = torch.empty(win.n_patches(8), device=DEV)
        s["loss"] = torch.empty(win.n_views, device=DEV)
        s["g_rgb"], s["g_pm"] = torch.empty_like(d["target"]), torch.empty_like(d["prior"])
        s["pose"] = torch.zeros(win.n_views, 6, device=DEV)
    if kind == "grad":
        s["leaves"] = [p.requires_grad_(True) for p in params]
        s["xi"] = torch.zeros(win.n_views, 6, device=DEV, requires_grad=True)
    return s


def run(s):
    kind = s["kind"]
    if kind == "pnp":
        T, count, mask, scores, T_n = pnp_ransac(s["X"], s["uv"], s["cam"], s["samples"], s["cfg"], T_ak=s["T_ak"],
                                                 ctx=s["ctx"])
        return {"T": T, "inliers": count, "mask": mask, "scores": scores, "T_n": T_n}
    rast = s["rast"]
    if kind == "align":
        rast.align_scale_into(s["Xr"], s["Xp"], s["result"], s["mask"], s["cfg"])
        rast.replace_pointmap_into(s["Xr"], s["Xp"], s["result"], s["hat"], s["replaced"])
        V = s["win"].n_views
        return {"scale": s["result"].view(torch.float64).view(V, 3)[:, 0],
                "counts": s["result"].view(torch.int32).view(V, 6)[:, 2:5], "hat": s["hat"],
                "replaced": s["replaced"]}
    params = s["params"]
    if kind == "track":
        out = s["out"]
        rast.forward_into(params, out, s["fs"])
        rast.window_loss_into(out["rgb"], s["target"], out["pointmap"], s["prior"], 8, 0.98, s["scale"], s["loss"],
                              s["g_rgb"], s["g_pm"])
        s["pose"].zero_()
        rast.pose_backward_into(params, out, {"rgb": s["g_rgb"], "pointmap": s["g_pm"]}, s["fs"], s["pose"])
        return {"out": out, "scale": s["scale"], "loss": s["loss"], "pose": s["pose"]}
    if kind == "map":
        step = s["step"]
        if step.graph is not None:
            step.replay()
        else:
            step.run()
        rast.iso_loss_into(params, 10.0, s["iso"], step.grads["log_scales"])
        return {"out": step.out, "scale": step.scale, "loss": step.loss, "iso": s["iso"], "grads": step.grads,
                "pose": step.pose_grad}
    if kind == "render":
        return rast.forward(params)[0]
    if kind == "grad":
        for t in (*s["leaves"], s["xi"]):
            t.grad = None
        images = rasterize(rast, *s["leaves"], s["xi"])
        torch.autograd.backward(images, [s["up"][k] for k in ("rgb", "depth", "alpha", "pointmap")])
        return {"out": dict(zip(("rgb", "depth", "alpha", "pointmap"), images)),
                "grads": {k: t.grad for k, t in zip(NAMES, s["leaves"])}, "pose": s["xi"].grad}
    rast.forward_into(params, s["out"], s["fs"])
    iou, oc, count = rast.covisibility(s["fs"])
    return {"out": s["out"], "iou": iou, "oc": oc, "count": count, "median": rast.median_depth(s["out"]["depth"])}


def work(case):
    """Bytes read and written once, and operations of the definition: 29 per composited fragment of
    the render and 64 of its backward.  Fragments are estimated from the density of the scene (about
    120 a visible Gaussian until a pixel saturates at about 95: 12.5 a pixel at 160x120 with 2k, 95 in
    the 8-view window)."""
    kind = case["kind"]
    if kind == "pnp":
        return {"bytes": 21.0 * case["n"] + 28.0 * case["hypotheses"], "flops": 30.0 * case["n"] * case["hypotheses"]}
    cams = _cams(case)
    P = float(sum(c.width * c.height for c in cams))
    if kind == "align":
        return {"bytes": P * (36 + 4 * case["mask"]), "flops": 60 * P}
    n = float(case["n"])
    frags = P * min(95.0, (120.0 if case["scene"] == "screen" else 70.0) * n * len(cams) / P)
    flops = {"render": 29, "keyframe": 29}.get(kind, 93) * frags
    per_px = {"render": 32, "keyframe": 32, "track": 56, "map": 56, "grad": 64}[kind]
    return {"bytes": 56 * n * (2 if kind in ("map", "grad") else 1) + per_px * P, "flops": flops}


# ---- the same results in float64 ---------------------------------------------------------------

NEAR, AMIN, AMAX, TMIN, EPS2D, CLAMP = 0.2, 1.0 / 255.0, 0.99, 1e-4, 0.3, 1.3


def _skew(p):
    o = torch.zeros_like(p[0])
    return torch.stack([o, -p[2], p[1], p[2], o, -p[0], -p[1], p[0], o]).view(3, 3)


def _project64(params, T12, xi, cam, frame):
    """Records [n][14] = (u, v, conic xx xy yy, opacity, colour 3, z, point 3, visible), the depth key
    and the half extents of the support."""
    means, ls, q, logit, rgb = params
    M = T12.double().view(3, 4)
    R, t = M[:, :3] + _skew(xi[3:]) @ M[:, :3], M[:, 3] + _skew(xi[3:]) @ M[:, 3] + xi[:3]
    m = R @ means + t[:, None]
    x, y, z = m
    vis = z.detach() > float(np.float32(NEAR))
    z1 = torch.where(vis, z, torch.ones_like(z))
    w, a, b, c = q / q.norm(dim=0)
    Rq = torch.stack([1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                      2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                      2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)]).view(3, 3, -1)
    A = (R[:, :, None, None] * Rq[None]).sum(1) * torch.exp(ls)[None]  # W Rq diag(s): [3][3][n]
    lx, ly = CLAMP * cam.width / (2 * cam.fx), CLAMP * cam.height / (2 * cam.fy)
    tx, ty = (x / z1).clamp(-lx, lx), (y / z1).clamp(-ly, ly)
    r0 = cam.fx / z1 * (A[0] - tx * A[2])  # the rows of J W Rq diag(s)
    r1 = cam.fy / z1 * (A[1] - ty * A[2])
    sxx, sxy, syy = (r0 * r0).sum(0) + EPS2D, (r0 * r1).sum(0), (r1 * r1).sum(0) + EPS2D
    det = sxx * syy - sxy * sxy
    al = torch.sigmoid(logit)
    vis = vis & (al.detach() >= float(np.float32(AMIN)))
    pt = m if frame else means
    rec = torch.stack([cam.fx * x / z1 + cam.cx, cam.fy * y / z1 + cam.cy, syy / det, -sxy / det, sxx / det, al,
                       *rgb, z, *pt], dim=1)
    ext = torch.sqrt(2 * torch.log((al / AMIN).clamp(min=1.0)) * torch.stack([sxx, syy])).detach()
    return rec, vis, ext


def _tiles64(rec, vis, ext, cam):
    """Tile lists in (float32 depth, index) order: the record of each pair, each tile's first, its length."""
    tw, th = -(-cam.width // 16), -(-cam.height // 16)
    with torch.no_grad():
        lo = torch.ceil(rec[:, :2] - ext.T - 0.01)
        hi = torch.floor(rec[:, :2] + ext.T + 0.01)
        size = torch.tensor([cam.width - 1, cam.height - 1], device=DEV)
        live = vis & (hi >= 0).all(1) & (lo <= size).all(1) & torch.isfinite(lo).all(1) & torch.isfinite(hi).all(1)
        idx = torch.nonzero(live).flatten()
        idx = idx[torch.sort(rec[idx, 9].float(), stable=True).indices]
        t0 = (lo[idx].clamp(min=0) // 16).long()
        t1 = (torch.minimum(hi[idx], size) // 16).long()
        nx, ny = (t1 - t0 + 1).unbind(1)
        owner = torch.repeat_interleave(torch.arange(idx.numel(), device=DEV), nx * ny)
        k = torch.arange(owner.numel(), device=DEV) - (torch.cumsum(nx * ny, 0) - nx * ny)[owner]
        tile = (t0[owner, 1] + k // nx[owner]) * tw + t0[owner, 0] + k % nx[owner]
        order = torch.sort(tile, stable=True)
        count = torch.bincount(tile, minlength=tw * th)
        return idx[owner[order.indices]], torch.cumsum(count, 0) - count, count


def _composite64(rec, lists, cam, frame, up=None, marks=None):
    """Images [8][H][W] (rgb, depth, alpha, point) of one view; with up (their upstream gradients, the
    same shape) the gradient of sum(up * images) with respect to rec instead."""
    pair, first, count = lists
    H, W = cam.height, cam.width
    tw = -(-W // 16)
    img = torch.zeros(8, H, W, dtype=torch.float64, device=DEV)
    grad = torch.zeros_like(rec) if up is not None else None
    px = torch.arange(256, device=DEV)
    by_size = torch.sort(count, descending=True).indices
    sizes = count[by_size].cpu().numpy()
    a, n_tiles = 0, int((sizes > 0).sum())
    while a < n_tiles:
        L = int(sizes[a])
        b = min(n_tiles, a + max(1, (12 if up is not None else 24) * 1_000_000 // (256 * L)))
        tiles = by_size[a:b]
        a = b
        k = torch.arange(L, device=DEV)[None]
        inside = k < count[tiles][:, None]
        r = pair[(first[tiles][:, None] + k).clamp(max=pair.numel() - 1)]
        x = (tiles % tw)[:, None] * 16 + px % 16
        y = (tiles // tw)[:, None] * 16 + px // 16
        on = (x < W) & (y < H)
        E = rec.detach()[r]  # [tiles][L][13]
        E.requires_grad_(up is not None)
        dx = x[:, :, None] - E[:, None, :, 0]
        dy = y[:, :, None] - E[:, None, :, 1]
        e = E[:, None, :, 2] * dx * dx + 2 * E[:, None, :, 3] * dx * dy + E[:, None, :, 4] * dy * dy
        al = (E[:, None, :, 5] * torch.exp(-0.5 * e)).clamp(max=AMAX)
        al = torch.where((al.detach() >= AMIN) & inside[:, None, :] & on[:, :, None], al, torch.zeros_like(al))
        lt = torch.log1p(-al)
        after = torch.cumsum(lt, 2)
        keep = after.detach() >= math.log(TMIN)
        w = torch.where(keep, al * torch.exp(after - lt), torch.zeros_like(al))
        if marks is not None:
            marks[r[((w.amax(1) > 0) & inside)]] = True
        v = torch.bmm(w, E[:, :, 6:13].contiguous())  # rgb, z, point
        alpha = 1 - torch.exp((lt * keep).sum(2))
        pt = v[:, :, 4:]
        if frame == 2:
            ray = torch.stack([(x - cam.cx) / cam.fx, (y - cam.cy) / cam.fy, torch.ones_like(x)], 2)
            pt = v[:, :, 3:4] * ray
        o = torch.cat([v[:, :, :4], alpha[:, :, None], pt], 2)
        xs, ys = x[on], y[on]
        if up is None:
            img[:, ys, xs] = o[on].T
        else:
            (o[on] * up[:, ys, xs].T).sum().backward()
            grad.index_add_(0, r.flatten(), torch.where(inside[:, :, None], E.grad, torch.zeros_like(E)).flatten(0, 1))
    return img if up is None else grad


def _patches64(X, patch):
    """[C][H][W] -> [patches][C][patch * patch], zero-padded, in row-major patch order."""
    C, h, w = X.shape
    ph, pw = -(-h // patch), -(-w // patch)
    Z = torch.zeros(C, ph * patch, pw * patch, dtype=X.dtype, device=X.device)
    Z[:, :h, :w] = X
    return Z.view(C, ph, patch, pw, patch).permute(1, 3, 0, 2, 4).reshape(ph * pw, C, -1)


def _loss64(img, target, prior):
    """Per-patch scale, loss and the upstream gradient of the images, one view."""
    _, h, w = img.shape
    a, b = _patches64(img[5:], 8), _patches64(prior, 8)
    den = (b * b).sum((1, 2))
    s = torch.where(den > 0, (a * b).sum((1, 2)) / den.clamp(min=1e-300), torch.ones_like(den))
    full = s.view(-(-h // 8), -(-w // 8)).repeat_interleave(8, 0).repeat_interleave(8, 1)[:h, :w]
    dp, dg = img[:3] - target, img[5:] - full * prior
    n = 3.0 * h * w
    up = torch.zeros_like(img)
    up[:3], up[5:] = 0.98 / n * dp.sign(), 0.02 / n * dg.sign()
    return s, 0.98 * dp.abs().sum() / n + 0.02 * dg.abs().sum() / n, up


def _planes(packed, cams, channels):
    o = 0
    for c in cams:
        k = channels * c.width * c.height
        yield packed[o:o + k].double().view(channels, c.height, c.width)
        o += k


def _images(imgs):
    return {"rgb": _packed([i[:3] for i in imgs]), "depth": _packed([i[3] for i in imgs]),
            "alpha": _packed([i[4] for i in imgs]), "pointmap": _packed([i[5:] for i in imgs])}


def _exact_render(case, d):
    kind, cams, frame = case["kind"], d["cams"], case.get("frame", 1)
    leaves = [p.detach().double().requires_grad_(True) for p in d["params"]]
    xi = torch.zeros(len(cams), 6, dtype=torch.float64, device=DEV, requires_grad=True)
    imgs, scale, loss, marks, ups = [], [], [], [], {}
    for k, v in d.get("up", {}).items():
        ups[k] = list(_planes(v, cams, 3 if k in ("rgb", "pointmap") else 1))
    targets = list(_planes(d["target"], cams, 3)) if "target" in d else None
    priors = list(_planes(d["prior"], cams, 3)) if "prior" in d else None
    for v, cam in enumerate(cams):
        rec, vis, ext = _project64(leaves, d["T"][v], xi[v], cam, frame)
        lists = _tiles64(rec, vis, ext, cam)
        mark = torch.zeros(case["n"], dtype=torch.bool, device=DEV) if kind == "keyframe" else None
        with torch.no_grad():
            imgs.append(_composite64(rec, lists, cam, frame, marks=mark))
        marks.append(mark)
        if kind in ("track", "map"):
            s, lv, up = _loss64(imgs[-1], targets[v], priors[v])
            scale.append(s)
            loss.append(lv)
        elif kind == "grad":
            up = torch.cat([ups["rgb"][v], ups["depth"][v], ups["alpha"][v], ups["pointmap"][v]])
        else:
            continue
        g = _composite64(rec, lists, cam, frame, up=up)
        # Records that no list holds may be infinite or undefined: they have no gradient.
        torch.where(vis[:, None], rec, torch.zeros_like(rec)).backward(g)
    out = _images(imgs)
    if kind == "render":
        return out
    if kind == "track":
        return {"out": out, "scale": torch.cat(scale), "loss": torch.stack(loss), "pose": xi.grad}
    if kind == "keyframe":
        M = torch.stack(marks).double()
        inter, size = M @ M.T, M.sum(1)
        return {"out": out, "iou": inter / (size[:, None] + size[None] - inter),
                "oc": inter / torch.minimum(size[:, None], size[None]), "count": None,
                "median": torch.stack([torch.sort(i[3][i[3] > 0]).values[((i[3] > 0).sum() - 1) // 2] for i in imgs])}
    grads = {k: t.grad for k, t in zip(NAMES, leaves)}
    if kind == "grad":
        return {"out": out, "grads": grads, "pose": xi.grad}
    with torch.no_grad():
        s = torch.exp(leaves[1])
        dev = s - s.mean(0, keepdim=True)
        sg = dev.sign()
        grads["log_scales"] = grads["log_scales"] + 10.0 * (sg - sg.mean(0, keepdim=True)) * s
        iso = 10.0 * dev.abs().sum().view(1)
    return {"out": out, "scale": torch.cat(scale), "loss": torch.stack(loss), "iso": iso, "grads": grads,
            "pose": xi.grad}


def _exact_align(case, d):
    scales, hats = [], []
    masks = list(_planes(d["mask"], d["cams"], 1)) if d["mask"] is not None else None
    for v, (Xr, Xp) in enumerate(zip(_planes(d["Xr"], d["cams"], 3), _planes(d["Xp"], d["cams"], 3))):
        valid = _patches64(masks[v] if masks else torch.ones_like(Xr[:1]), case["patch"])[:, 0]
        nr, np_ = (_patches64(X.norm(dim=0, keepdim=True), case["patch"])[:, 0] for X in (Xr, Xp))
        n = valid.sum(1).clamp(min=1.0)
        mu = [(x * valid).sum(1) / n for x in (nr, np_)]
        sd = [torch.sqrt(((x - m[:, None]) ** 2 * valid).sum(1) / n) for x, m in zip((nr, np_), mu)]
        z = [(x - m[:, None]) / s.clamp(min=1e-300)[:, None] for x, m, s in zip((nr, np_), mu, sd)]
        cp = ((z[0] - z[1]).abs() < float(np.float32(0.1))) & (valid > 0) & ((sd[0] > 0) & (sd[1] > 0))[:, None]
        s, d3 = torch.ones((), dtype=torch.float64, device=DEV), float(np.float32(0.3))
        for _ in range(3):
            cand = ((mu[0] - s * mu[1]).abs() < d3 * s * mu[1]) & ((sd[0] - s * sd[1]).abs() < d3 * s * sd[1])
            use = cp & (cand & (valid.sum(1) > 0))[:, None]
            if use.any():
                s = nr[use].sum() / np_[use].sum()
        scales.append(s)
        h = s * Xp
        hats.append(torch.where((Xr - h).norm(dim=0) <= float(np.float32(0.15)) * h.norm(dim=0), Xr, h))
    return {"scale": torch.stack(scales), "counts": None, "hat": _packed(hats), "replaced": None}


def _exact_pnp(case, d):
    cam = d["cam"]
    X, uv = d["X"].double().cpu(), d["uv"].double().cpu()
    fx, fy = float(np.float32(cam.fx)), float(np.float32(cam.fy))
    f, c = torch.tensor([[fx], [fy]], dtype=torch.float64), torch.tensor([[cam.cx], [cam.cy]], dtype=torch.float64)
    idx = d["samples"].long().cpu()
    P, x = X[:, idx].permute(1, 2, 0), ((uv - c) / f)[:, idx].permute(1, 2, 0)  # [H][6][3], [H][6][2]
    cen = P.mean(1, keepdim=True)
    s = math.sqrt(3.0) / (P - cen).norm(dim=2).mean(1)
    Xh = torch.cat([s[:, None, None] * (P - cen), torch.ones_like(P[:, :, :1])], 2)
    O = torch.zeros_like(Xh)
    A = torch.cat([torch.cat([Xh, O, -x[:, :, :1] * Xh], 2), torch.cat([O, Xh, -x[:, :, 1:] * Xh], 2)], 1)
    N = torch.linalg.svd(A).Vh[:, -1].view(-1, 3, 4)
    M = s[:, None, None] * N[:, :, :3]
    p4 = N[:, :, 3] - (M @ cen.transpose(1, 2))[:, :, 0]
    sign = torch.where(torch.linalg.det(M) < 0, -1.0, 1.0)
    U, S, Vt = torch.linalg.svd(sign[:, None, None] * M)
    R, t = U @ Vt, sign[:, None] * p4 / S.mean(1)[:, None]

    def inliers(R, t):
        Y = R @ X + t[..., None]
        r = f * Y[..., :2, :] / Y[..., 2:, :] + c - uv
        return (Y[..., 2, :] > 0) & ((r * r).sum(-2) < 9.0), Y, r

    score = torch.stack([inliers(R[h], t[h])[0].sum() for h in range(R.shape[0])])
    best = int(torch.nonzero(score == score.max())[0])
    R, t = R[best], t[best]
    for _ in range(2):
        use = inliers(R, t)[0]
        for _ in range(10):
            _, Y, r = inliers(R, t)
            Y, r = Y[:, use], r[:, use]
            iz, o = 1 / Y[2], torch.zeros_like(Y[2])
            J = []
            for g in (torch.stack([fx * iz, o, -fx * Y[0] * iz * iz]), torch.stack([o, fy * iz, -fy * Y[1] * iz * iz])):
                J.append(torch.cat([g, torch.linalg.cross(Y, g, dim=0)]))
            J, e = torch.cat(J, 1), r.reshape(-1)
            Hm = J @ J.T
            Hm = Hm + 1e-9 * torch.trace(Hm) / 6 * torch.eye(6, dtype=torch.float64)
            step = torch.linalg.solve(Hm, -(J @ e))
            G = torch.zeros(4, 4, dtype=torch.float64)
            G[:3, :3], G[:3, 3] = _skew(step[3:]), step[:3]
            G = torch.linalg.matrix_exp(G)
            R, t = G[:3, :3] @ R, G[:3, :3] @ t + G[:3, 3]
    T = torch.cat([R, t[:, None]], 1)
    ak = torch.cat([d["T_ak"].double().cpu().view(3, 4), torch.tensor([[0.0, 0, 0, 1]], dtype=torch.float64)])
    return {"T": T, "inliers": None, "mask": None, "scores": None, "T_n": (T @ ak).reshape(-1)}


def exact(case, seed):
    if case["kind"] not in ("pnp", "align"):
        pixels = sum(c.width * c.height for c in _cams(case))
        if pixels > 4_000_000 or case["n"] * len(_cams(case)) > 10_000_000:
            return None  # the float64 composite of a large window takes too long
    d = _inputs(case, seed)
    return {"pnp": _exact_pnp, "align": _exact_align}.get(case["kind"], _exact_render)(case, d)
