"""CPU tests of the numbers that decide which triangles the fast stage-1 tests may drop, taken from the host
plan itself: a draw's margin (reach), the pixels a unit of length projects to (scale), what a strip's sphere gets on
top (grow); and of the launch shapes of captured graphs, which follow sizes and options alone."""
import numpy as np
import pytest
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W
from plan_draws import INTERIOR, plan_draws

f32 = np.float32


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(f32)


def _row(A, v):
    return _fma(A[0], v[:, 0], _fma(A[1], v[:, 1], _fma(A[2], v[:, 2], np.full(len(v), A[3], f32))))


def _rcp(w, ulps):
    r = (1.0 / w.astype(np.float64)).astype(f32)
    return np.where(ulps > 0, np.nextafter(r, f32(np.inf)), np.where(ulps < 0, np.nextafter(r, f32(-np.inf)), r)).astype(f32)


def _snapped(D, v, half):
    """Exact path: window positions snapped to 1/256 px, in pixels, [n, 2]."""
    w = _row(D["A"][8:], v)
    zi = (1.0 / w.astype(np.float64)).astype(f32)
    return np.stack([np.rint(np.float64(_fma((_row(D["A"][4 * k:], v) * zi).astype(f32), half[k], half[k])) * 256.0) / 256.0
                     for k in (0, 1)], 1)


def _in_ball(rng, n, c, r):
    d = rng.normal(size=(n, 3))
    d *= r * rng.uniform(0, 1, (n, 1)) ** (1 / 3) / np.linalg.norm(d, axis=1, keepdims=True)
    return c + d


def _mesh(pos, inst=None, triangles=4):
    pos = np.asarray(pos, np.float32)
    return api.GpuMesh(torch.from_numpy(pos), torch.zeros(triangles, 3, dtype=torch.int32), inst, W.bounding_sphere(pos))


def _draws(size, seed, count, **options):
    """(draw, bounding sphere, view) of random placements: near and far, meshes up to ten radii off their origin."""
    rng = np.random.default_rng(seed)
    for _ in range(count):
        off = rng.normal(size=3) * 10 ** rng.uniform(-1, 1)
        pos = _in_ball(rng, 8, off, 1.0)
        depth = 10 ** rng.uniform(0.1, 2.5)
        scale = 10 ** rng.uniform(-3, 0)
        t = np.array([[rng.uniform(-0.6, 0.6) * depth, rng.uniform(-0.4, 0.4) * depth, -depth]])
        R = W.random_rotations(rng, 1)
        inst = W.instance_matrices(R, np.array([scale]), t - scale * (R[0] @ off)[None])
        view = W.View(W.camera((0.0, 0.0, 0.0), (0.0, 0.0, -1.0), aspect=1.0), W.NEAR, size, max(1, size * 9 // 16))
        m = _mesh(pos, inst)
        for D in plan_draws([m], [view], **options)[0]:
            yield rng, D, m.bsphere.astype(np.float64), view


@pytest.mark.parametrize("flags", [0, api.FLAG_NO_FAST_INTERIOR])
@pytest.mark.parametrize("size", [1, 17, 256, 1920, 16384])
def test_reach_covers_the_fast_positions(size, flags):
    """Window positions as the kernels compute them, from the prescaled rows or the exact transform with a
    reciprocal one ulp off, lie within reach - 1/2 of the snapped ones."""
    seen = {True: 0, False: 0}
    for rng, D, bs, view in _draws(size, size, 400, flags=flags):
        half = (f32(view.width / 2), f32(view.height / 2))
        v = _in_ball(rng, 24, bs[:3], bs[3]).astype(f32)
        w = _row(D["A"][8:], v)
        x, y = _row(D["A"][0:], v), _row(D["A"][4:], v)
        ok = (w >= f32(view.near)) & (abs(x) <= 2 * w) & (abs(y) <= 2 * w)
        v, w = v[ok], w[ok]
        exact = _snapped(D, v, half)
        r = _rcp(w, rng.integers(-1, 2, len(w)))
        margin = float(D["reach"]) - 0.5
        interior = bool(D["view"] & INTERIOR)
        for k in (0, 1):
            general = np.float64(_fma((_row(D["A"][4 * k:], v) * r).astype(f32), half[k], half[k]))
            if interior:
                fast = np.float64((_row(D["R"][4 * k:], v) * r).astype(f32))
                assert (abs(fast - exact[:, k]) <= margin).all(), (size, abs(fast - exact[:, k]).max(), margin)
            assert (abs(general - exact[:, k]) <= margin).all(), (size, abs(general - exact[:, k]).max(), margin)
        seen[interior] += len(v)
    assert seen[not flags] > 1000, seen


@pytest.mark.parametrize("size", [64, 1920, 16384])
def test_scale_and_grow_cover_strip_spheres(size):
    """The box around a strip sphere's projected centre, scale times its radius plus grow to each side, holds the
    snapped window positions of every point of the sphere with the half pixel and the margin to spare."""
    seen = loose = 0
    for rng, D, bs, view in _draws(size, 100 + size, 500):
        if not D["view"] & INTERIOR:
            continue
        half = (f32(view.width / 2), f32(view.height / 2))
        if D["scale"] == 0:
            loose += 1
            continue
        assert D["scale"] > 0 and D["grow"] >= D["reach"]
        for _ in range(6):
            r = bs[3] * 10 ** rng.uniform(-3, -0.3)
            c = _in_ball(rng, 1, bs[:3], bs[3] - r)[0].astype(f32)
            v = np.concatenate([_in_ball(rng, 12, c, r), c + r * np.eye(3), c - r * np.eye(3)])
            v = v[np.linalg.norm(v - bs[:3], axis=1) <= bs[3]].astype(f32)
            # as strip_sphere gives it: rounded, then inflated by 2^-10
            rs = f32(f32(np.linalg.norm(v.astype(np.float64) - c, axis=1).max()) * f32(1.0 + 1.0 / 1024.0))
            exact = _snapped(D, v, half)
            rw = _rcp(_row(D["A"][8:], c[None]), rng.integers(-1, 2, 1))
            ext = np.float64(_fma(D["scale"], rs, D["grow"]))
            for k in (0, 1):
                centre = (_row(D["R"][4 * k:], c[None]) * rw).astype(np.float64)[0]
                off = abs(exact[:, k] - centre).max()
                assert off <= ext - 0.5, (size, off, ext)
            seen += len(v)
    assert seen > 5000 and loose > 0, (seen, loose)


def test_shapes_of_large_launches():
    """What the defaults choose for a launch of many work items: strips of 4, spheres for draws of tiny
    triangles and boxes for the others of the same mesh, more than 32 draws per work item."""
    rng = np.random.default_rng(0)
    pos, _ = W.uv_sphere(6, 12, 1.0)
    n = 300
    inst = W.instance_matrices(W.random_rotations(rng, n), 10 ** rng.uniform(-2, -0.5, n), rng.uniform(-0.8, 0.8, (n, 3)))
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0)), W.NEAR, 1000, 1000)
    draws, shape = plan_draws([_mesh(pos, inst, triangles=2100000)], [view])
    assert shape["tpt_multi"] == 4 and shape["spheres"] == 1 and shape["draws_per_item"] == 128
    scale = draws["scale"]
    assert (scale < 0).any() and (scale > 0).any()
    assert (draws["view"][scale > 0] & INTERIOR).all()
    small = plan_draws([_mesh(pos, inst, triangles=300)], [view])[1]
    assert small["tpt_multi"] == 2 and small["draws_per_item"] == 8


@pytest.mark.parametrize("opts", [{}, dict(s1_mode=3), dict(s1_draws_per_item=5), dict(s1_multi_tris_per_thread=8)])
def test_graph_shapes_follow_sizes_alone(opts):
    """Whatever the cameras cull, a captured graph's kernels and grid stay the same; only the draws per work
    item, which the frame's header carries, and the choice between the two captured variants may change."""
    rng = np.random.default_rng(1)
    pos, _ = W.uv_sphere(6, 12, 1.0)
    meshes = [_mesh(pos, W.instance_matrices(W.random_rotations(rng, n), rng.uniform(0.01, 0.05, n), rng.uniform(-2, 2, (n, 3))), t)
              for n, t in ((1, 900000), (400, 40000), (7, 2000), (1, 12))]
    fixed = set()
    counts = set()
    for z in (40.0, 6.0, 2.1, -9.0, 200.0):
        views = [W.View(W.camera((0.1 * i, 0.0, z), (0.1 * i, 0.0, z - 1.0)), W.NEAR, 300, 200) for i in range(3)]
        _, s = plan_draws(meshes, views, graph=True, **opts)
        fixed.add((s["tpt_single"], s["tpt_multi"], s["read_first"], s["max_items"]))
        counts.add(s["draws"])
    assert len(counts) > 2 and len(fixed) == 1, (counts, fixed)


def test_single_draw_launch_reads_by_density():
    """What the single-draw launch reads before its atomics follows the triangles per pixel: nothing below a
    quarter, samples from there on, every key from 32."""
    pos, _ = W.uv_sphere(6, 12, 1.0)
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0)), W.NEAR, 200, 100)
    for triangles, reads in ((4999, 0), (5000, 2), (639999, 2), (640000, 3)):
        for graph in (False, True):
            assert plan_draws([_mesh(pos, None, triangles)], [view], graph)[1]["read_first"] == reads, triangles


@pytest.mark.parametrize("n_meshes", [1, 2, 25, 40])
@pytest.mark.parametrize("n_views", [1, 2, 7])
def test_draw_records_are_cache_lines(n_meshes, n_views):
    """The records start at a multiple of their 128 bytes in the descriptor block, whatever comes before them."""
    pos, _ = W.uv_sphere(6, 12, 1.0)
    views = [W.View(W.camera((0.0, 0.0, 3.0 + i), (0.0, 0.0, 0.0)), W.NEAR, 64, 64) for i in range(n_views)]
    assert plan_draws([_mesh(pos)] * n_meshes, views)[1]["offset"] % 128 == 0


@pytest.mark.parametrize("instances,per_item", [(600, 64), (100, 8), (3000, 128)])
def test_vertex_sharing_items_keep_more_draws(instances, per_item):
    """Mode 3 deduplicates an item's vertices first, so its items keep more draws than the strip kernel's."""
    rng = np.random.default_rng(instances)
    pos, _ = W.uv_sphere(6, 12, 1.0)
    inst = W.instance_matrices(W.random_rotations(rng, instances), np.full(instances, 0.01), rng.uniform(-0.5, 0.5, (instances, 3)))
    view = W.View(W.camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0)), W.NEAR, 1000, 1000)
    mesh = _mesh(pos, inst, triangles=131072)
    assert plan_draws([mesh], [view], s1_mode=3)[1]["draws_per_item"] == per_item
    assert plan_draws([mesh], [view])[1]["draws_per_item"] <= per_item
