"""GPU test of the multi-draw launch as the defaults shape it for many work items: strips of 4, up to 128 draws
per item, spheres and boxes in one launch, against the exact-only mode bit for bit (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W
from plan_draws import plan_draws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["strips", "mixed"])
@pytest.mark.parametrize("instances,views", [(150, 1), (130, 2), (40, 3)])
def test_spheres_and_boxes_in_one_launch(order, instances, views):
    rng = np.random.default_rng(instances)
    pos, idx = W.uv_sphere(1024, 1024, 1.0)
    if order == "mixed":                    # a few work items that are no strips
        a = rng.choice(len(idx), 400, replace=False)
        idx[np.sort(a)] = idx[a]
    t = np.stack([rng.uniform(-s, s, instances) for s in (1.9, 1.3, 1.0)], 1)
    inst = W.instance_matrices(W.random_rotations(rng, instances), 10 ** rng.uniform(-2.3, -0.1, instances), t)
    mesh = W.Mesh(pos, idx, inst=inst, bsphere=W.bounding_sphere(pos))
    vs = [W.View(W.camera((0.2 * i, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=1.4), W.NEAR, 420 + 17 * i, 300) for i in range(views)]
    gm = api.GpuMesh.from_host(mesh)
    draws, shape = plan_draws([gm], vs, graph=True)
    assert shape["tpt_multi"] == 4 and shape["draws_per_item"] > 32 and shape["spheres"] == 1
    assert (draws["scale"] < 0).any() and (draws["scale"] > 0).any()
    with api.Context() as c, api.Context(s1_mode=1) as exact:
        for _ in range(2):
            for a, b in zip(c.rasterize_batched([gm], vs), exact.rasterize_batched([gm], vs)):
                assert torch.equal(a, b)
        small = c.compress(gm)
        for a, b in zip(c.rasterize_batched([small], vs), exact.rasterize_batched([small], vs)):
            assert torch.equal(a, b)
