"""Host-side check of the benchmark's launch shapes: options that a context leaves open (0) are reported as the
launch chooses them, so that the rooflines name and count the kernels that run."""
import importlib.util
import os

import numpy as np
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _mesh(triangles, n, scale):
    rng = np.random.default_rng(n)
    pos, _ = W.uv_sphere(6, 12, 1.0)
    inst = W.instance_matrices(W.random_rotations(rng, n), np.full(n, scale), rng.uniform(-0.5, 0.5, (n, 3)))
    return api.GpuMesh(torch.from_numpy(pos), torch.zeros(triangles, 3, dtype=torch.int32), inst, W.bounding_sphere(pos))


def test_open_options_name_the_kernels_that_run():
    b = _bench()
    gm = [_mesh(300000, 1, 0.5), _mesh(2100000, 300, 0.01), _mesh(100000, 2, 0.4)]
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0)), W.NEAR, 1000, 1000)
    opts = {n: 0 for n, _ in api.Options._fields_}
    opts.update(s1_block=64)
    h = {"name": "x", "shape": b.launch_shape(api, gm, [view], opts), "options": opts, "single": [], "multi_items": 630200000,
         "single_items": 300000, "stage_ms": {"stage1_multi": 2.0, "stage1_single": 1.0},
         "stats": {"strip_draws": 157500000, "strip_sphere_pass": 1000, "strip_union_pass": 100}}
    assert h["shape"] == {"single": 1, "multi": 4, "draws_per_item": 128, "strips": True, "spheres": True, "box_items": 200000}
    multi, single = b.stage1_rooflines(h)
    assert multi["kernel"].startswith("stage1_strips_kernel<4, true, false, 0>")
    assert single["kernel"].startswith("stage1_fast_kernel<64, 1, false, 0>")
    boxes = 50000
    assert multi["algorithmic_lane_ops"] == ((157500000 - boxes) * b.SPHERE_OPS + (boxes + 1000) * b.strip_draw_ops(4) +
                                             100 * 4 * b.box_ops(3) + 200000 * b.LONE_TRI_DRAW_OPS)
    fixed = dict(opts, s1_mode=4, s1_multi_tris_per_thread=8, s1_tris_per_thread=4)
    shape = b.launch_shape(api, gm, [view], fixed)
    assert (shape["single"], shape["multi"], shape["strips"], shape["spheres"]) == (4, 8, True, False)
