"""CPU tests of the launch shapes that the host plan chooses when the options leave them open, by the work
items it counts."""
import numpy as np
import pytest
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W


def _mesh(triangles, inst=None, sphere=False):
    pos = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0]], np.float32)
    return api.GpuMesh(torch.from_numpy(pos), torch.zeros(triangles, 3, dtype=torch.int32), inst,
                       W.bounding_sphere(pos) if sphere else None)


def _view(size=64, eye=(0.0, 0.0, 3.0)):
    return W.View(W.camera(eye, (0.0, 0.0, 0.0)), W.NEAR, size, size)


def _items(meshes, views, **opts):
    return api.plan(meshes, views, **opts)[2]["work_items"]


@pytest.mark.parametrize("triangles", [1, 255, 257, 699999, 700001, 7000001])
def test_single_strips_flag_takes_strips(triangles):
    """CURAST_FLAG_SINGLE_STRIPS with the triangles per lane left open: strips of 4 (64 lanes each) at every
    size, since one triangle per lane is no strip; given triangles per lane stay what they are."""
    m = [_mesh(triangles)]
    assert _items(m, [_view()], flags=api.FLAG_SINGLE_STRIPS) == -(-triangles // 256)
    for tpt in (1, 2, 8):
        assert _items(m, [_view()], flags=api.FLAG_SINGLE_STRIPS, s1_tris_per_thread=tpt) == -(-triangles // (64 * tpt))
    for off in (dict(flags=api.FLAG_SINGLE_STRIPS | api.FLAG_NO_STRIPS), dict(flags=api.FLAG_SINGLE_STRIPS, s1_mode=1)):
        assert _items(m, [_view()], **off) == _items(m, [_view()])
