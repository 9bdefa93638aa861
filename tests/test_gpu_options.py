"""GPU tests of the context's options: reading and setting them again changes nothing, and the autotuner
keeps the choices that are left to every launch (needs an MI355X)."""
import json

import numpy as np
import pytest
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu

OPEN = ("s1_tris_per_thread", "s1_multi_tris_per_thread", "s1_draws_per_item")


def _scene():
    """A mesh drawn once and one drawn 9 times, few enough that the launches' own shapes differ from 4
    triangles per lane and 64 draws per work item."""
    rng = np.random.default_rng(3)
    meshes = []
    for n in (1, 9):
        pos, idx = W.uv_sphere(24, 48, 0.4)
        inst = W.instance_matrices(W.random_rotations(rng, n), np.ones(n), rng.uniform(-0.8, 0.8, (n, 3)))
        meshes.append(W.Mesh(pos, idx, inst=inst, bsphere=W.bounding_sphere(pos)))
    return meshes, W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0)), W.NEAR, 200, 200)


@pytest.mark.parametrize("opts", [{}, dict(s1_multi_tris_per_thread=2), dict(s1_draws_per_item=3, s1_mode=4),
                                  dict(s1_tris_per_thread=8, flags=api.FLAG_NO_TINY_CULL)])
def test_setting_what_was_read_changes_nothing(opts):
    meshes, view = _scene()
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    expect = api.plan(gm, [view], **opts)[2]
    with api.Context(**opts) as c:
        first = c.options()
        c.set_options(**first)
        assert c.options() == first
        assert api.plan(gm, [view], **first)[2] == expect
        assert [first[k] for k in OPEN] == [opts.get(k, 0) for k in OPEN]


def test_autotuned_options_may_stay_open(tmp_path):
    """A cached choice of 0 leaves the choice open in the context that reads it."""
    meshes, view = _scene()
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    vis = torch.empty((view.height, view.width), dtype=torch.int64, device="cuda")
    path = tmp_path / "tune.jsonl"
    with api.Context() as c:
        c.autotune(gm, [view], [vis], cache_path=str(path))
    entry = json.loads(path.read_text())
    entry.update({k: 0 for k in OPEN}, s1_mode=0)
    path.write_text(json.dumps(entry) + "\n")
    with api.Context() as c:
        chosen = c.autotune(gm, [view], [vis], cache_path=str(path))
        assert [chosen[k] for k in OPEN] == [0, 0, 0]
        assert api.plan(gm, [view], **chosen)[2] == api.plan(gm, [view], s1_block=chosen["s1_block"])[2]
