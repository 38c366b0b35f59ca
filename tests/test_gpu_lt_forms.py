"""Which form of L^T a call takes (its launches, read from a captured graph), and its values there.

sl_apply_LT adds a member's terms in an LDS copy of its source grid where that
fits, else by a thread per pixel straight to memory.  Values against the FP64
oracle within 2 (terms + 4) u of the sum of absolute terms, as in the
operators' test (which explains the bound).
"""
import numpy as np
import pytest
import torch

import synthgen
from captured import kernel_launches
from oracle import lens as olens
from oracle import operators as oops

pytestmark = pytest.mark.gpu
DEV = "cuda"
U = {torch.float32: 2.0 ** -24, torch.float64: 2.0 ** -53}


def _call(nx, nsub, ns, dtype, ordered=False, check=()):
    import paper_1101_5803_amd as sl
    grid = sl.Grid(nx, nx, 4.0 / nx, nsub)
    G = synthgen.population(11, len(ns))
    img = np.random.default_rng(nx).standard_normal((len(ns), grid.J)).astype(np.float32).astype(np.float64)
    uv = sl.lens_trace(torch.tensor(G, device=DEV), grid, ns, 1.0)
    it = torch.tensor(img, dtype=dtype, device=DEV)
    call = lambda: (sl.apply_LT_ordered if ordered else sl.apply_LT)(uv, grid, ns, it)
    got = call().double().cpu().numpy()
    off = np.concatenate([[0], np.cumsum(np.square(ns))])
    for m in check:
        idx, w, inside = oops.bilinear_table(*olens.trace_image(G[m], nx, nx, grid.pix, nsub), ns[m], 1.0)
        if dtype == torch.float32:   # the fractions that the FP32 operator holds
            fx, fy = ((w[..., a] + w[..., 3]).astype(np.float32).astype(np.float64) for a in (1, 2))
            w = np.where(inside[..., None], np.stack([(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy], -1), 0.0)
        tab = (idx, w, inside)
        ref, ones = (oops.apply_LT(tab, v, ns[m] ** 2, nsub) for v in (img[m], np.abs(img[m])))
        cnt = np.bincount(np.asarray(idx).reshape(-1), minlength=ns[m] ** 2)
        bound = 2 * (cnt + 4) * U[dtype] * ones + 64 * ns[m] * U[torch.float64] * cnt * np.abs(img[m]).max()
        assert np.all(np.abs(got[off[m]:off[m + 1]] - ref) <= bound), m
    return kernel_launches(call)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_large_grid_has_a_thread_per_pixel(dtype):
    """A grid that LDS cannot hold: as many threads as pixels, not a few blocks that walk them."""
    (grid, block, lds) = _call(512, 1, [200], dtype, check=(0,))[-1]
    assert lds == 0 and grid[0] * block[0] >= 512 * 512


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ns", [(64, 64), (96, 99), (32, 142)])
def test_lds_copy_is_fp64(nx, ns, dtype):
    """ds_add_f32 takes several times as long as ds_add_f64, so both types add in FP64 copies."""
    (_, _, lds) = _call(nx, 2, [ns], dtype, check=(0,))[-1]
    assert lds == 8 * ns * ns


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_each_member_takes_its_own_form(dtype):
    """One grid past LDS among small ones: they keep their LDS form, whatever the order."""
    ns = [40] * 10 + [150] + [38] * 20
    launches = _call(64, 2, ns, dtype, check=(0, 10, 11, 30))
    assert sorted((g[1], lds > 0) for g, b, lds in launches if b[0] in (256, 512))[-2:] == [(1, False), (30, True)]
    # the ordered form's two binning passes, in the LDS and the memory form each
    bins = [(g[1], lds > 0) for g, b, lds in _call(64, 2, ns, dtype, ordered=True, check=(0, 10, 11, 30)) if b[0] == 512]
    assert sorted(bins) == [(1, False), (1, False), (30, True), (30, True)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_ordered_rows_of_every_length_on_a_sparse_grid(dtype):
    """A grid with more nodes than the image has subpixels takes a lane per row; bits as a wave per row."""
    import paper_1101_5803_amd as sl
    grid = sl.Grid(32, 32, 0.1, 2)
    rng = np.random.default_rng(4)
    uv = torch.full((1, 4096, 2), float("nan"), dtype=torch.float64)
    at = rng.permutation(4096)
    for cell, n in enumerate([1, 2, 7, 8, 9, 63, 64, 70, 511, 600]):   # cells two apart: no node has two cells
        k, at = at[:n], at[n:]
        uv[0, k, 0] = torch.tensor(2 * (cell % 4) + rng.uniform(0, 1, n))
        uv[0, k, 1] = torch.tensor(2 * (cell // 4) + rng.uniform(0, 1, n))
    uv = uv.to(DEV)
    img = torch.tensor(rng.standard_normal((1, 1024)), dtype=dtype, device=DEV)
    out, launches = {}, {}
    for ns in (12, 100):   # 144 nodes: a wave per row; 10000: sparse
        out[ns] = sl.apply_LT_ordered(uv, grid, [ns], img).reshape(ns, ns)
        nodes = kernel_launches(lambda: sl.apply_LT_ordered(uv, grid, [ns], img))
        launches[ns] = nodes[-1]
        assert [lds > 0 for _, block, lds in nodes if block[0] == 512] == [ns == 12] * 2   # the binning passes
    assert torch.equal(out[100][:12, :12], out[12]) and not out[100][12:].any() and not out[100][:, 12:].any()
    assert launches[12][0][0] * launches[12][1][0] == 64 * 144
    assert launches[100][0][0] * launches[100][1][0] < 2 * 10000
    _call(48, 1, [200], dtype, ordered=True, check=(0,))


def test_rows_of_a_small_grid_beside_a_sparse_one():
    """Lane or wave per row is each member's own choice: 3600 nodes (fewer than subpixels) beside 4900 and 22500."""
    (grid, block, _) = _call(32, 2, [70, 60, 150], torch.float64, ordered=True, check=(0, 1, 2))[-1]
    assert grid[0] * block[0] >= 64 * 3600
