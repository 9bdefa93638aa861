"""GPU test of the backward's per-tile table where as many vertices as a tile can have crowd into few of its
rows: every pixel its own triangle, vertex indices that agree in their low bits (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 16, 1024, 1025, 2049, 16384])
@pytest.mark.parametrize("channels", [1, 3, 8])
def test_crowded_tables(stride, channels):
    """A triangle per pixel, its vertices `stride` apart: 768 distinct vertices in each tile of 16 x 16."""
    w, h = 35, 18
    n = 3 * w * h
    rng = np.random.default_rng(stride + channels)
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=w / h), W.NEAR, w, h)
    half = 3.0 / np.reshape(view.vp, (4, 4))[1, 1]
    px, py = np.meshgrid(np.arange(w) + 0.5, np.arange(h) + 0.5)
    c = np.stack([(2 * px / w - 1) * half * w / h, (2 * py / h - 1) * half, 0 * px], 2).reshape(-1, 1, 3)
    d = half / h * np.array([[-0.7, -0.7, 0.0], [0.8, -0.6, 0.1], [0.0, 0.9, -0.1]])
    pos = np.zeros((n * stride, 3), np.float32)
    order = rng.permutation(n) * stride                     # which vertex sits where in the tile is random
    pos[order] = (c + d).reshape(-1, 3)
    mesh = W.Mesh(pos, order.reshape(-1, 3).astype(np.uint32), attrs=rng.normal(size=(len(pos), channels)).astype(np.float32))
    vis = O.rasterize([mesh], view)
    assert len(np.unique(vis)) == w * h
    g = rng.normal(size=(h, w, channels)).astype(np.float32)
    pss = O.project(mesh, view)
    ref = O.resolve_screen_backward_f64(vis, mesh.idx, 0, pss, mesh.attrs, g.astype(np.float64))
    gm = api.GpuMesh.from_host(mesh)
    tvis, tg, tp = torch.from_numpy(vis.view(np.int64)).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(pss).cuda()
    with api.Context() as ctx:
        for with_pos in (True, False):
            for one in (True, False):
                ga = torch.zeros_like(gm.attrs)
                gp = torch.zeros_like(gm.pos) if with_pos else None
                if one:
                    ctx.resolve_backward(tvis, gm.idx, tp, gm.attrs, tg, ga, gp)
                else:
                    ctx.resolve_backward_meshes([gm], view, tvis, [gm.attrs], tg, [ga], [gp] if with_pos else None)
                for got, want in ((ga, ref[0]), (gp, ref[1])):
                    if got is None:
                        continue
                    scale = np.maximum(np.abs(want), 1e-3 * np.sqrt(np.mean(want ** 2)) + 1e-30)
                    err = np.abs(got.cpu().numpy().astype(np.float64) - want) / scale
                    assert err.max() <= 1e-3, (stride, channels, with_pos, one, err.max())
