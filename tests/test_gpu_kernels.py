"""GPU tests of kernel variants at the sizes where they can go wrong: tile edges, remainders, channel
counts with and without a kernel of their own, short and long queues, small and large descriptor
blocks (needs an MI355X).  Visibility buffers must equal the oracle's, resolves agree within 1e-5,
gradients within the acceptance bound of the differentiable resolve (1e-3 of the value, floored at
1e-3 of the root mean square)."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import assert_resolve_close, assert_vis_equal
from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = api.Context()
    yield c
    c.close()


def _sphere_and_ground(lat, lon, channels, seed=0):
    """A sphere of 2 lat lon triangles on a ground quad that crosses the near plane."""
    rng = np.random.default_rng(seed)
    pos, idx = W.uv_sphere(lat, lon, 1.0)
    gpos = np.array([[-10, -1, -10], [10, -1, -10], [-10, -1, 10], [10, -1, 10]], np.float32)
    gidx = np.array([[0, 2, 1], [1, 2, 3]], np.uint32)
    return [W.Mesh(p, i, attrs=rng.normal(size=(len(p), channels)).astype(np.float32), bsphere=W.bounding_sphere(p))
            for p, i in ((pos, idx), (gpos, gidx))]


def _view(width, height):
    return W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), aspect=width / height), W.NEAR, width, height)


def _assert_grads(got, ref, what):
    scale = np.maximum(np.abs(ref), 1e-3 * np.sqrt(np.mean(ref ** 2)) + 1e-30)
    err = np.abs(got.cpu().numpy().astype(np.float64) - ref) / scale
    assert err.max() <= 1e-3, f"{what}: {err.max()}"


@pytest.mark.parametrize("size", [(1, 1), (15, 17), (33, 16), (130, 95)])
@pytest.mark.parametrize("channels", [1, 2, 3, 4, 5, 8, 11, 16])
def test_resolve_and_backward_by_channel_count(ctx, size, channels):
    """Resolve, differentiable resolve and both backward forms, with vertices that hundreds of pixels
    of a tile share (the ground) and vertices of single pixels (the sphere)."""
    meshes = _sphere_and_ground(40, 81, channels)
    view = _view(*size)
    rng = np.random.default_rng(9)
    vis = O.rasterize(meshes, view)
    tvis = torch.from_numpy(vis.view(np.int64)).cuda()
    gout = rng.normal(size=(view.height, view.width, channels)).astype(np.float32)
    tg = torch.from_numpy(gout).cuda()
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    out = ctx.resolve(gm, view, tvis, [g.attrs for g in gm]).cpu().numpy()
    assert_resolve_close(out, O.resolve(meshes, view, vis, [m.attrs for m in meshes]), "resolve")
    one = O.rasterize(meshes[:1], view)          # one mesh: descriptors straight from the argument
    got = ctx.resolve(gm[:1], view, torch.from_numpy(one.view(np.int64)).cuda(), [gm[0].attrs]).cpu().numpy()
    assert_resolve_close(got, O.resolve(meshes[:1], view, one, [meshes[0].attrs]), "resolve of one mesh")
    bases = O.id_bases(meshes)
    pss = [O.project(m, view) for m in meshes]
    ref = [O.resolve_screen_backward_f64(vis, m.idx, int(b), p, m.attrs, gout.astype(np.float64))
           for m, b, p in zip(meshes, bases, pss)]
    for with_pos in (True, False):
        ga = [torch.zeros_like(g.attrs) for g in gm]
        gp = [torch.zeros_like(g.pos) for g in gm] if with_pos else None
        ctx.resolve_backward_meshes(gm, view, tvis, [g.attrs for g in gm], tg, ga, gp)
        for m in range(2):
            _assert_grads(ga[m], ref[m][0], f"attrs of mesh {m}")
            if with_pos:
                _assert_grads(gp[m], ref[m][1], f"positions of mesh {m}")
            ga1 = torch.zeros_like(gm[m].attrs)
            gp1 = torch.zeros_like(gm[m].pos) if with_pos else None
            tp = torch.from_numpy(pss[m]).cuda()
            ctx.resolve_backward(tvis, gm[m].idx, tp, gm[m].attrs, tg, ga1, gp1, id_base=int(bases[m]))
            _assert_grads(ga1, ref[m][0], f"one-mesh form, attrs of mesh {m}")
            if with_pos:
                _assert_grads(gp1, ref[m][1], f"one-mesh form, positions of mesh {m}")
    assert_resolve_close(ctx.resolve_screen(tvis, gm[0].idx, torch.from_numpy(pss[0]).cuda(), gm[0].attrs).cpu().numpy(),
                         O.resolve_screen(vis, meshes[0].idx, 0, pss[0], meshes[0].attrs), "screen resolve")


@pytest.mark.parametrize("k,channels,size", [(2, 1, (3, 2)), (2, 5, (17, 9)), (2, 16, (40, 31)), (4, 3, (5, 7)),
                                             (4, 8, (33, 18))])
def test_supersampled_tiles(ctx, k, channels, size):
    """Supersampling at sizes around its tiles of 8 x 8 (2 x 2 samples) and 4 x 4 pixels."""
    meshes = _sphere_and_ground(20, 41, channels)
    view = _view(size[0] * k, size[1] * k)
    vis = O.rasterize(meshes, view)
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    out = ctx.resolve(gm, view, torch.from_numpy(vis.view(np.int64)).cuda(), [g.attrs for g in gm], samples_per_axis=k)
    ref = O.resolve_supersampled(meshes, view, vis, [m.attrs for m in meshes], k)
    assert_resolve_close(out.cpu().numpy(), ref, f"{k} x {k}")


@pytest.mark.parametrize("n_meshes", [1, 2, 7, 8, 9, 10, 16, 17, 40])
def test_descriptor_block_sizes(ctx, n_meshes):
    """Frames and resolves whose descriptors travel in the kernel argument (few meshes) and through
    device memory (many), with instances among them."""
    rng = np.random.default_rng(n_meshes)
    meshes = []
    for i in range(n_meshes):
        pos, idx = W.uv_sphere(6, 9, 0.3)
        inst = W.instance_matrices(W.random_rotations(rng, 1 + i % 3), np.ones(1 + i % 3),
                                   rng.uniform(-1.5, 1.5, (1 + i % 3, 3)))
        meshes.append(W.Mesh(pos, idx, inst=inst, attrs=rng.random((len(pos), 3), dtype=np.float32),
                             bsphere=W.bounding_sphere(pos)))
    view = _view(150, 111)
    gm = [api.GpuMesh.from_host(m) for m in meshes]
    for _ in range(2):
        vis = ctx.rasterize_meshes(gm, view)
        ref = O.rasterize(meshes, view)
        assert_vis_equal(api.as_uint64(vis), ref, f"{n_meshes} meshes")
        out = ctx.resolve(gm, view, vis, [g.attrs for g in gm]).cpu().numpy()
        assert_resolve_close(out, O.resolve(meshes, view, ref, [m.attrs for m in meshes]), f"{n_meshes} meshes")


@pytest.mark.parametrize("triangles", [1, 63, 64, 65, 700])
@pytest.mark.parametrize("opts", [{}, dict(s2_waves=4), dict(medium_px=1), dict(medium_px=1, q3_capacity=9)])
def test_stage2_and_stage3_queue_lengths(triangles, opts):
    """Queues of stage 2 shorter and longer than its wavefronts, and stage-3 tile lists of many parts."""
    rng = np.random.default_rng(triangles)
    c = rng.uniform(-1.2, 1.2, (triangles, 1, 3)) * (1, 1, 0.5)
    pos = (c + rng.normal(0, 0.25, (triangles, 3, 3))).reshape(-1, 3).astype(np.float32)
    m = W.Mesh(pos, np.arange(3 * triangles, dtype=np.uint32).reshape(-1, 3))
    view = _view(321, 203)
    with api.Context(small_px=1, **opts) as c:
        vis = c.rasterize_meshes([api.GpuMesh.from_host(m)], view)
        assert_vis_equal(api.as_uint64(vis), O.rasterize([m], view), f"{triangles} triangles {opts}")


@pytest.mark.parametrize("vertices,triangles", [(3, 1), (4, 2), (1023, 341), (1366, 2049), (70001, 33333)])
def test_compression_ranges(ctx, vertices, triangles):
    """Index range, bounding box, packing and quantization at remainders of their 16-byte loads, word
    groups and pair stores, against the oracle bit for bit."""
    rng = np.random.default_rng(vertices)
    pos = rng.normal(size=(vertices, 3)).astype(np.float32) * (1, 1e-3, 50)
    idx = rng.integers(vertices // 3, vertices, (triangles, 3)).astype(np.uint32)
    m = W.Mesh(pos.astype(np.float32), idx)
    small = ctx.compress(api.GpuMesh.from_host(m)).compressed
    index_min, bits, words = O.compress_indices(m.idx)
    lo, step = O.position_box(m.pos)
    assert (small.index_min, small.index_bits) == (index_min, bits)
    assert np.array_equal(small.lo, lo) and np.array_equal(small.step, step)
    assert np.array_equal(small.packed.cpu().numpy().view(np.uint32), words)
    q = small.qpos.cpu().numpy().view(np.uint16)
    assert q[-1] == 0 and np.array_equal(q[:-1].reshape(-1, 3), O.quantize_positions(m.pos, lo, step))


@pytest.mark.parametrize("order", ["strips", "shuffled", "mixed"])
@pytest.mark.parametrize("lat,scale,instances", [(4, 0.5, 2), (24, 0.3, 9), (96, 0.05, 40), (128, 0.01, 300)])
def test_multi_draw_launch_shapes(ctx, order, lat, scale, instances):
    """The multi-draw launch as the library shapes it by itself: strips of 8 with spheres for tiny
    triangles, boxes otherwise, few and many draws per work item, odd triangle counts, meshes without a
    bounding sphere, work items that are not strips throughout."""
    rng = np.random.default_rng(lat)
    pos, idx = W.uv_sphere(lat, 2 * lat + 1, 1.0)
    idx = idx[:-1]
    if order == "shuffled":
        idx = idx[rng.permutation(len(idx))]
    elif order == "mixed":
        swap = rng.choice(len(idx), len(idx) // 50 + 2, replace=False)
        idx[np.sort(swap)] = idx[swap]
    t = np.stack([rng.uniform(-1.8, 1.8, instances), rng.uniform(-1.2, 1.2, instances),
                  rng.uniform(-3, 3.2, instances)], axis=1)
    inst = W.instance_matrices(W.random_rotations(rng, instances), rng.uniform(0.5, 2, instances) * scale, t)
    view = _view(233, 170)
    for sphere in (True, False):
        m = W.Mesh(pos, idx, inst=inst, bsphere=W.bounding_sphere(pos) if sphere else None)
        vis = ctx.rasterize_meshes([api.GpuMesh.from_host(m)], view)
        assert_vis_equal(api.as_uint64(vis), O.rasterize([m], view), f"{order} {lat} {instances} sphere {sphere}")


@pytest.mark.parametrize("n_views", [1, 16, 24])
@pytest.mark.parametrize("instances", [26, 27, 301, 2500])
def test_descriptors_from_pinned_memory(instances, n_views):
    """Frames in flight whose descriptors lie past the kernel argument: the first launch reads them from
    pinned memory (views in the argument) or a copy uploads them (too many views)."""
    pos, idx = W.uv_sphere(4, 8, 1.0)
    views = [_view(16 + i, 20) for i in range(n_views)]
    rng = np.random.default_rng(instances)
    with api.Context(flags=api.FLAG_NO_GRAPH) as c:
        frames = []
        for _ in range(5):
            t = np.stack([rng.uniform(-2, 2, instances), rng.uniform(-1.5, 1.5, instances),
                          rng.uniform(-3, 3, instances)], axis=1)
            inst = W.instance_matrices(W.random_rotations(rng, instances), rng.uniform(0.02, 0.2, instances), t)
            m = W.Mesh(pos, idx, inst=inst)
            g = api.GpuMesh.from_host(m)
            frames.append((m, g, c.rasterize_batched([g], views) if n_views > 1 else [c.rasterize_meshes([g], views[0])]))
        for k, (m, _, vis) in enumerate(frames):
            for i in range(0, n_views, 7):
                assert_vis_equal(api.as_uint64(vis[i]), O.rasterize([m], views[i]), f"frame {k} view {i}")
