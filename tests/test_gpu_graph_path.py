"""GPU test of batched frames along a camera path (needs an MI355X): whatever the cameras cull, however large
the triangles get, later frames replay what the first one captured, and every frame equals the eager one."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PATH = r'''
import sys
import numpy as np, torch
from paper_2604_21749_amd import api, workloads as W
rng = np.random.default_rng(5)
meshes = []
for n, lat in ((1, 40), (1500, 60), (12, 24)):
    pos, idx = W.uv_sphere(lat, 2 * lat, 1.0)
    t = rng.uniform(-2, 2, (n, 3))
    inst = W.instance_matrices(W.random_rotations(rng, n), rng.uniform(0.01, 0.03, n), t)
    meshes.append(W.Mesh(pos, idx, inst=inst, bsphere=W.bounding_sphere(pos)))
with api.Context() as graph, api.Context(flags=api.FLAG_NO_GRAPH) as eager:
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    # everything in view and far, close up, one instance left, nothing left, back again
    eyes = [(0, 0, 40.0), (0, 0, 6.0), (0, 0, 2.1), (1.9, 1.9, 2.05), (0, 0, -9.0), (0, 0, 40.0), (0, 0, 200.0)]
    for k, e in enumerate(eyes):
        views = [W.View(W.camera(e, (e[0], e[1], e[2] - 1.0)), W.NEAR, 161, 120 + 9 * i) for i in range(3)]
        print("frame", k, file=sys.stderr, flush=True)
        got, ref = graph.rasterize_batched(gm, views), eager.rasterize_batched(gm, views)
        for a, b in zip(got, ref):
            assert torch.equal(a, b), k
print("path ok")
'''


def test_camera_path_replays_one_capture():
    env = dict(os.environ, CURAST_LOG="1", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PATH], capture_output=True, text=True, env=env, cwd=ROOT, timeout=100)
    assert r.returncode == 0 and "path ok" in r.stdout, r.stderr[-2000:]
    parts = re.split(r"^frame \d+$", r.stderr, flags=re.M)
    captures = [len(re.findall("captured a frame graph", p)) for p in parts[1:]]
    assert len(captures) == 7 and captures[0] >= 1 and not any(captures[1:]), captures
