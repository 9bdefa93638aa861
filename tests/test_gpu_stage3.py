"""GPU tests of stage 3's two ways to split the screen among workgroups, at the numbers of tiles and
workgroups where it changes from one to the other, against the oracle bit for bit (needs an MI355X)."""
import numpy as np
import pytest

import oracle as O
from helpers import assert_vis_equal
from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


def _triangles(n, size, seed):
    rng = np.random.default_rng(seed)
    c = rng.uniform(-1.2, 1.2, (n, 1, 3)) * (1, 1, 0.5)
    return W.Mesh((c + rng.normal(0, size, (n, 3, 3))).reshape(-1, 3).astype(np.float32),
                  np.arange(3 * n, dtype=np.uint32).reshape(-1, 3))


@pytest.mark.parametrize("size,blocks", [((321, 203), 1), ((321, 203), 31), ((321, 203), 32), ((321, 203), 0),
                                         ((1000, 700), 1), ((1000, 700), 2), ((1000, 700), 175), ((65, 64), 2)])
@pytest.mark.parametrize("n,spread", [(1, 3.0), (40, 1.5), (300, 0.2)])
def test_tiles_and_workgroups(size, blocks, n, spread):
    """24, 176 and 2 tiles over few and many workgroups (0: the default): quarters up to three rounds of them,
    whole tiles from there on, also where one workgroup has more than 64 tiles; lists of one part and of many,
    and tiles without any."""
    mesh = _triangles(n, spread, 7 * n + blocks)
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=size[0] / size[1]), W.NEAR, *size)
    with api.Context(medium_px=1, small_px=1, s3_blocks=blocks) as c:
        vis = c.rasterize_meshes([api.GpuMesh.from_host(mesh)], view)
        assert_vis_equal(api.as_uint64(vis), O.rasterize([mesh], view), f"{size} {blocks} {n}")


@pytest.mark.parametrize("blocks", [1, 3, 0])
def test_tiles_of_several_views(blocks):
    mesh = _triangles(60, 0.8, 3)
    views = [W.View(W.camera((0.3 * i, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=1.2), W.NEAR, 70 + 64 * i, 90 + 50 * i)
             for i in range(5)]
    with api.Context(medium_px=1, small_px=1, s3_blocks=blocks) as c:
        for _ in range(2):
            for i, vis in enumerate(c.rasterize_batched([api.GpuMesh.from_host(mesh)], views)):
                assert_vis_equal(api.as_uint64(vis), O.rasterize([mesh], views[i]), f"view {i}")
