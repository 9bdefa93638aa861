"""GPU test of the resolves at every channel count, bit for bit the same through every form that gives the
same values, and against the oracle (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import assert_resolve_close
from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels", range(1, 17))
def test_every_channel_count(channels):
    """Plain resolve of one and of two meshes and the differentiable one; the last channel of the last
    pixel ends where the buffer does, so a store past it would show in the guard behind."""
    rng = np.random.default_rng(channels)
    w, h = 61, 47
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=w / h), W.NEAR, w, h)
    meshes = []
    for k, lat in enumerate((9, 30)):
        pos, idx = W.uv_sphere(lat, 2 * lat, 0.9)
        pos = (pos + np.array([1.1 * k - 0.5, 0.0, 0.3 * k], np.float32)).astype(np.float32)
        meshes.append(W.Mesh(pos, idx, attrs=rng.normal(size=(len(pos), channels)).astype(np.float32)))
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    with api.Context() as ctx:
        for n in (1, 2):
            vis = ctx.rasterize_meshes(gm[:n], view)
            host = api.as_uint64(vis)
            room = torch.full((w * h * channels + 64,), 7.0, dtype=torch.float32, device="cuda")
            out = room[:w * h * channels].view(h, w, channels)
            ctx.resolve(gm[:n], view, vis, [g.attrs for g in gm[:n]], out=out)
            assert_resolve_close(out.cpu().numpy(), O.resolve(meshes[:n], view, host, [m.attrs for m in meshes[:n]]),
                                 f"{n} meshes, {channels} channels")
            assert (room[w * h * channels:] == 7.0).all()
            if n == 1:
                screen = ctx.resolve_screen(vis, gm[0].idx, ctx.project(gm[0], view), gm[0].attrs)
                assert torch.equal(screen, out)
