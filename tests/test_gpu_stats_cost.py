"""GPU test of frames that count (CURAST_FLAG_STATS): their launches do not spend their time on the counters
(needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


def _frame_ms(mesh, view, flags):
    with api.Context(flags=api.FLAG_TIMING | flags) as c:
        vis = c.rasterize_meshes([mesh], view)
        best = 1e9
        for _ in range(8):
            c.reset_stage_times()
            c.rasterize_meshes([mesh], view, out=vis)
            torch.cuda.synchronize()
            best = min(best, c.stage_times()["frame"])
        return best, vis


def test_counting_frames_of_many_work_items():
    """16 to 25 thousand work items: one workgroup each, adding to the same counters, took ten times a plain
    frame; the bound leaves twice the room that the counting itself takes."""
    rng = np.random.default_rng(2)
    pos, idx = W.uv_sphere(256, 256, 1.0)
    n = 600
    inst = W.instance_matrices(W.random_rotations(rng, n), np.full(n, 0.02), rng.uniform(-1, 1, (n, 3)))
    gm = api.GpuMesh.from_host(W.Mesh(pos, idx, inst=inst, bsphere=W.bounding_sphere(pos)))
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=16 / 9), W.NEAR, 1920, 1080)
    plain, ref = _frame_ms(gm, view, 0)
    counting, vis = _frame_ms(gm, view, api.FLAG_STATS)
    assert torch.equal(vis, ref)
    assert counting < 6 * plain, (counting, plain)
