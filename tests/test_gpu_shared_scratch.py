"""Calls that share a context's scratch do not move it under one another's captured graphs.

The isotropic regulariser, the covisibility and the median depth use one scratch buffer.  A graph
holds its address, so it may not be allocated again when a later call needs more of it: the
regulariser captured in a graph has to replay correctly after the first median and covisibility
of the same Rasterizer, for any number of views.  After ``reserve`` none of them (and no forward
or backward) allocates, so each can be captured without a first call outside the capture.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import binding  # noqa: E402
from paper_2507_03737_amd.render import Rasterizer, Window  # noqa: E402
from paper_2507_03737_amd.scenes import Camera  # noqa: E402

from . import gpu_util as U  # noqa: E402

pytestmark = pytest.mark.gpu


def lower_median(x):
    x = np.sort(x[x > 0])
    return x[(len(x) - 1) // 2] if len(x) else 0.0


@pytest.mark.parametrize("views", [1, 7, 8, 32])
def test_regulariser_graph_after_first_median(views):
    U.log(f"[gpu] shared scratch, {views} views")
    rng = np.random.default_rng(views)
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    n = 3000
    params = (f32(np.stack([rng.uniform(-1, 1, n), rng.uniform(-1, 1, n), rng.uniform(2, 5, n)])),
              f32(rng.uniform(-4, -2, (3, n))), f32(rng.normal(size=(4, n))), f32(rng.normal(size=n)),
              f32(rng.uniform(0, 1, (3, n))))
    cams = [Camera(40 + v, 31, 40.0, 40.0, 20.0 + v / 2, 15.5) for v in range(views)]
    T = f32(np.tile([1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0], (views, 1)))
    rast = Rasterizer(Window(cams, T), n, binding.RasterConfig(mark_visible=1), max_pairs=1 << 18)
    rast.reserve()
    out, fs = rast.new_outputs(), rast.new_frame_state()
    iou, oc = (torch.empty(views, views, dtype=torch.float64, device="cuda") for _ in range(2))
    loss, grad, med = torch.empty(1, device="cuda"), torch.zeros(3, n, device="cuda"), torch.empty(views, device="cuda")
    grads, pose = rast.zero_grads(params), torch.empty(views, 6, device="cuda")

    def iso():
        grad.zero_()
        rast.iso_loss_into(params, 0.5, loss, grad)

    def frame():
        rast.forward_into(params, out, fs)
        rast.backward_into(params, out, {"rgb": out["rgb"]}, fs, grads, pose, overwrite=True)
        binding.median_depth(rast.ctx, rast.win.c(), out["depth"], med, binding.stream_handle())
        binding.covisibility(rast.ctx, rast.win.c(), n, fs, iou, oc, None, binding.stream_handle())

    torch.cuda.synchronize()
    graphs = []
    for work in (iso, frame):  # nothing was called before: a call that allocates fails here
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            work()
        graphs.append(graph)
    for k in range(3):
        params[1].add_(0.25 * k)  # the next replays see other scales
        s = np.exp(params[1].cpu().numpy().astype(np.float64))
        want = 0.5 * np.abs(s - s.mean(axis=0)).sum()
        eager = rast.median_depth(out["depth"]) if k else None
        for graph in graphs:
            graph.replay()
        filler = [torch.full((1 << 16,), 7.0, device="cuda") for _ in range(4)]  # later allocations
        graphs[0].replay()
        torch.cuda.synchronize()
        assert abs(float(loss) - want) <= 1e-6 * want
        depth = out["depth"].cpu().numpy()
        planes = [depth[a:b] for a, b in zip(rast.win.pix_off, rast.win.pix_off[1:])]
        assert np.array_equal(med.cpu().numpy(), np.float32([lower_median(d) for d in planes]))
        assert np.all(np.diag(iou.cpu().numpy()) == 1.0) and (eager is None or eager.shape == (views,))
        assert all(float(g.abs().sum()) > 0 for g in grads.values()) and len(filler) == 4
