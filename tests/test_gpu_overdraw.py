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
    """Triangles of less and of more than 1.5 px, one layer and nine, in every order."""
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


@pytest.mark.parametrize("size", [(64, 64), (61, 33), (200, 5)])
def test_boxes_past_the_view_without_tiny_culling(size):
    """Triangles that miss the view past its corners, where no single side culls them: without tiny culling they
    reach the small rasterizer with an empty box, which holds no pixel to sample."""
    rng = np.random.default_rng(size[0])
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=size[0] / size[1]), W.NEAR, *size)
    half = 3.0 / np.reshape(view.vp, (4, 4))[1, 1]
    c = rng.choice([-1.0, 1.0], (6000, 1, 2)) * np.array([half * size[0] / size[1], half])
    d = rng.uniform(-0.06, 0.06, (6000, 3, 2)) + 0.03 * np.sign(c)
    pos = np.concatenate([c + d, rng.uniform(-0.1, 0.1, (6000, 3, 1))], 2).reshape(-1, 3).astype(np.float32)
    mesh = W.Mesh(pos, np.arange(18000, dtype=np.uint32).reshape(-1, 3))
    ref = O.rasterize([mesh], view)
    gm = api.GpuMesh.from_host(mesh)
    guard = torch.full((3 * size[1], size[0]), -1, dtype=torch.int64, device="cuda")
    for flags in (0, api.FLAG_NO_TINY_CULL, api.FLAG_NO_TINY_CULL | api.FLAG_STATS):
        for mode in (0, 1):
            guard.fill_(-1)
            with api.Context(flags=flags, s1_mode=mode) as ctx:
                ctx.rasterize_meshes([gm], view, out=guard[size[1]:2 * size[1]])
            assert_vis_equal(api.as_uint64(guard[size[1]:2 * size[1]]), ref, f"{size} {flags} {mode}")
            assert (guard[:size[1]] == -1).all() and (guard[2 * size[1]:] == -1).all()
