"""The host plan's draws as the kernels read them (curast_internal_plan_draws), for the tests."""
import ctypes as C

import numpy as np

from paper_2604_21749_amd import api

DRAW = np.dtype([("A", "f4", 12), ("R", "f4", 8), ("id_base", "u8"), ("view", "u4"), ("mesh", "u4"), ("scale", "f4"),
                 ("grow", "f4"), ("wmax", "f4"), ("hmax", "f4"), ("vis", "u8"), ("near", "f4"), ("reach", "f4")])
assert DRAW.itemsize == 128
INTERIOR = 0x80000000


def plan_draws(meshes, views, graph=False, **options):
    """(records, shape dict) of the draws that survive the cull, in order."""
    keep = []
    arr = api._mesh_array(meshes, keep, check=False)
    vis = (C.c_uint64 * len(views))()
    vs = (api.ViewStruct * len(views))()
    for i, v in enumerate(views):
        vs[i] = api._view_struct(v.vp, v.near, v.width, v.height, None)
        vs[i].visbuffer = C.addressof(vis) + 8 * i
    room = sum(m.num_instances for m in meshes) * len(views)
    draws = np.zeros(room, DRAW)
    shape = (C.c_uint64 * 8)()
    opt = api.Context._options(options)
    f = api.lib().curast_internal_plan_draws
    f.argtypes = [C.c_void_p, C.c_uint32, C.c_void_p, C.c_uint32, C.c_void_p, C.c_int, C.c_void_p, C.c_uint64, C.c_void_p]
    rc = f(arr, len(meshes), vs, len(views), C.byref(opt), int(graph), draws.ctypes.data, room, shape)
    assert rc == api.OK, rc
    names = ("draws", "tpt_single", "tpt_multi", "draws_per_item", "spheres", "read_first", "max_items",
             "offset")
    shape = dict(zip(names, map(int, shape)))
    return draws[:shape["draws"]], shape
