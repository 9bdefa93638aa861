"""GPU test of layered scenes, where the small rasterizer decides triangle by triangle whether to read the
stored key before its atomics: the visibility buffer equals the oracle's whatever it decides (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import assert_vis_equal
from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


def _layers(cell, layers, order, view, jitter):
    """`layers` grids of `cell` px over the view, tilted against one another so that they intersect."""
    half = 3.0 / view.vp[1][1] if np.ndim(view.vp) == 2 else 3.0 / view.vp.reshape(4, 4)[1][1]
    nx, ny = int(view.width / cell) + 1, int(view.height / cell) + 1
    gy, gx = np.meshgrid(np.linspace(-half, half, ny + 1), np.linspace(-half, half, nx + 1) * view.width / view.height,
                         indexing="ij")
    i = (np.arange(ny)[:, None] * (nx + 1) + np.arange(nx)).reshape(-1)
    q = np.stack([i, i + 1, i + nx + 1, i + 1, i + nx + 2, i + nx + 1], 1).reshape(-1, 3)
    rng = np.random.default_rng(layers)
    pos = np.concatenate([np.stack([gx, gy, 0.01 * k + jitter * rng.normal() * gx], 2).reshape(-1, 3) for k in range(layers)])
    idx = np.stack([q + k * gx.size for k in range(layers)])
    if order == "front":
        idx = idx[::-1]
    elif order == "mixed":
        idx = idx.transpose(1, 0, 2)
    return W.Mesh(pos.astype(np.float32), np.ascontiguousarray(idx.reshape(-1, 3)).astype(np.uint32))


@pytest.mark.parametrize("cell", [0.9, 1.7, 1.8, 3.4, 3.6, 5.3])
@pytest.mark.parametrize("layers,order,jitter", [(1, "back", 0.0), (9, "back", 0.0), (9, "front", 0.01), (9, "mixed", 0.03)])
def test_layers(cell, layers, order, jitter):
    """Triangles just below and above 1.5 and 6 px, one layer and nine, in every order."""
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=203 / 157), W.NEAR, 203, 157)
    mesh = _layers(cell, layers, order, view, jitter)
    ref = O.rasterize([mesh], view)
    assert (ref != O.EMPTY).mean() > 0.9
    gm = api.GpuMesh.from_host(mesh)
    for opts in ({}, dict(s1_mode=1), dict(flags=api.FLAG_STATS), dict(flags=api.FLAG_NO_EARLY_OUT),
                 dict(flags=api.FLAG_EARLY_OUT_ALL), dict(flags=api.FLAG_SINGLE_STRIPS)):
        with api.Context(**opts) as c:
            assert_vis_equal(api.as_uint64(c.rasterize_meshes([gm], view)), ref, f"{cell} {layers} {order} {opts}")
            vis = torch.empty((view.height, view.width), dtype=torch.int64, device="cuda")
            c.rasterize_noalloc(gm.pos, gm.idx, view.vp, view.near, view.width, view.height, vis)
            assert_vis_equal(api.as_uint64(vis), ref, f"{cell} {layers} {order} {opts}, allocation-free")
