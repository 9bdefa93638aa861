"""GPU test of the stage-1 overflow pass with few stage-2 wavefronts (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import assert_vis_equal
from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


def _frame_ms(mesh, view, **opts):
    with api.Context(flags=api.FLAG_TIMING, **opts) as c:
        vis = c.rasterize_meshes([mesh], view)
        best = 1e9
        for _ in range(5):
            c.reset_stage_times()
            c.rasterize_meshes([mesh], view, out=vis)
            torch.cuda.synchronize()
            best = min(best, c.stage_times()["frame"])
        return best, api.as_uint64(vis)


@pytest.mark.parametrize("waves", [1, 64, 0])
def test_overflow_pass_does_not_depend_on_the_stage2_wavefronts(waves):
    """A full queue is drained by the whole chip whatever s2_waves is: with 1 or 16 workgroups for it, as many as
    stage 2's, it took 10 to 150 times as long (the bound of 4 leaves room for stage 2 itself)."""
    pos, idx = W.uv_sphere(512, 1024, 1.0)
    mesh = W.Mesh(pos, idx)
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=16 / 9), W.NEAR, 1280, 720)
    gm = api.GpuMesh.from_host(mesh)
    ref_ms, _ = _frame_ms(gm, view, small_px=1, q2_capacity=100)
    ms, vis = _frame_ms(gm, view, small_px=1, q2_capacity=100, s2_waves=waves)
    assert_vis_equal(vis, O.rasterize([mesh], view), f"s2_waves {waves}")
    assert ms < 4 * ref_ms, (waves, ms, ref_ms)
