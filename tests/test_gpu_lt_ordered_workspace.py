"""The ordered L^T takes any workspace from one member's size up, with the same bits."""
import ctypes

import numpy as np
import pytest
import torch

import synthgen

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("members_held", [1, 2, 3])
def test_smaller_workspaces(members_held):
    import paper_1101_5803_amd as sl
    from paper_1101_5803_amd import _lib as B
    L = B.lib()
    ns = [30, 21, 30, 9, 17]
    grid = sl.Grid(40, 36, 0.1, 2)
    uv = sl.lens_trace(torch.tensor(synthgen.population(11, len(ns)), device=DEV), grid, ns, 1.0)
    img = torch.tensor(np.random.default_rng(1).standard_normal((len(ns), grid.J)), device=DEV)
    want = sl.apply_LT_ordered(uv, grid, ns, img)
    g, arr = grid.c(), B.i32_array(ns)
    size = L.sl_apply_LT_ordered_workspace_size(ctypes.byref(g), arr, members_held)   # ns[0] is the largest
    guard = 4096
    ws = torch.full((size + guard,), 171, dtype=torch.uint8, device=DEV)
    out = torch.full_like(want, float("nan"))
    def run(nbytes):
        return L.sl_apply_LT_ordered(B.SL_F64, B.ptr(uv), len(ns), ctypes.byref(g), arr, B.ptr(img), B.ptr(out),
                                     B.ptr(ws), nbytes, B.stream_handle())
    assert run(size) == 0, L.sl_last_error()
    assert torch.equal(out, want) and torch.all(ws[size:] == 171)
    if members_held == 1:
        assert run(size - 4) == -1 and b"workspace too small" in L.sl_last_error()
