"""Argument checks of the resolves that need no GPU: a list of attributes shorter than the mesh list is
refused before the library, which reads one pointer per mesh, sees it."""
import types

import numpy as np
import pytest
import torch

from paper_2604_21749_amd import api
from paper_2604_21749_amd import workloads as W


def _mesh(triangles):
    return api.GpuMesh(torch.zeros(3, 3), torch.zeros(triangles, 3, dtype=torch.int32))


@pytest.fixture
def calls(monkeypatch):
    """A context whose library records the pointer arrays it is given; device checks are left out."""
    seen = []

    def resolve(h, arr, M, view, ptrs, *rest):
        seen.append((M, list(ptrs)))
        return api.OK
    monkeypatch.setattr(api, "lib", lambda: types.SimpleNamespace(
        curast_resolve=resolve, curast_resolve_supersampled=lambda h, arr, M, view, ss, ptrs, *r: resolve(h, arr, M, view, ptrs)))
    monkeypatch.setattr(api, "_check_cuda", lambda *a, **k: None)
    monkeypatch.setattr(api, "_stream", lambda dev=None: 0)
    ctx = api.Context.__new__(api.Context)
    ctx._h = None
    return ctx, seen


@pytest.mark.parametrize("samples", [1, 2])
@pytest.mark.parametrize("triangles,given,ok", [((1, 1), 1, False), ((1, 1, 0), 1, False), ((1, 0, 1), 2, False),
                                                ((1, 0), 1, True), ((1, 1), 2, True), ((1,), 2, True)])
def test_resolve_with_fewer_attrs_than_meshes(calls, samples, triangles, given, ok):
    ctx, seen = calls
    meshes = [_mesh(t) for t in triangles]
    attrs = [torch.zeros(3, 4) for _ in range(given)]
    view = W.View(np.eye(4, dtype=np.float32), 0.1, 8, 8)
    vis = torch.zeros(8, 8, dtype=torch.int64)
    if not ok:
        with pytest.raises(ValueError, match="attrs"):
            ctx.resolve(meshes, view, vis, attrs, samples_per_axis=samples)
        assert not seen
        return
    ctx.resolve(meshes, view, vis, attrs, samples_per_axis=samples)
    (M, ptrs), = seen
    assert M == len(meshes) <= len(ptrs)
    assert ptrs[:min(given, M)] == [a.data_ptr() for a in attrs[:M]] and not any(ptrs[given:M])
