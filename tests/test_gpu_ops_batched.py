"""The stand-alone operators at the edges of their tiles, batches and LDS forms, against the FP64 oracle.

Tolerances: a sum of n rounded products with rounded terms is within
(n + 4) u sum |terms| of its exact value (u the unit roundoff, 4 for the
rounded weights and inputs), evaluated per output with the oracle's operator
on absolute values; twice that allows for the oracle's own rounding in FP64.
FP32 operators hold the bilinear fractions in FP32, so the oracle's table is
given those fractions (1 - f of a rounded f is not within a relative u).
"""
import numpy as np
import pytest
import torch

import synthgen
from oracle import lens as olens
from oracle import operators as oops

pytestmark = pytest.mark.gpu
DEV = "cuda"
U = {torch.float32: 2.0 ** -24, torch.float64: 2.0 ** -53}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("K,ny,nx,n", [(1, 5, 3, 2), (3, 64, 8, 1), (7, 65, 9, 3), (9, 63, 31, 2), (17, 64, 32, 1),
                                       (15, 130, 33, 1), (15, 128, 128, 33), (63, 70, 41, 1), (63, 20, 300, 9)])
def test_blur_tiles(dtype, K, ny, nx, n):
    import paper_1101_5803_amd as sl
    rng = np.random.default_rng(K + nx)
    P = rng.uniform(0.1, 1.0, (K, K)) / K ** 2      # asymmetric: a flipped or shifted tap shows
    x = rng.standard_normal((n, ny, nx)).astype(np.float32).astype(np.float64)
    xt = torch.tensor(x, dtype=dtype, device=DEV)
    pt = torch.tensor(P, device=DEV)
    for got, op in ((sl.apply_B(pt, xt), oops.apply_B), (sl.apply_BT(pt, xt), oops.apply_BT)):
        got = got.double().cpu().numpy()
        for i in {0, n // 2, n - 1}:
            bound = 2 * (K * K + 4) * U[dtype] * op(P, np.abs(x[i])) + 1e-300
            assert np.all(np.abs(got[i] - op(P, x[i])) <= bound)


def test_blur_keeps_non_finite_values_local():
    import paper_1101_5803_amd as sl
    x = np.ones((70, 50))
    x[30, 20], x[5, 44] = np.inf, np.nan
    P = np.full((5, 5), 0.04)
    for dtype in U:
        for op in (sl.apply_B, sl.apply_BT):
            got = op(torch.tensor(P, device=DEV), torch.tensor(x, dtype=dtype, device=DEV)).cpu().numpy()
            hit = np.zeros(x.shape, bool)
            hit[28:33, 18:23] = True
            hit[3:8, 42:47] = True
            assert np.all(np.isfinite(got) == ~hit)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ny,nsub,ns", [
    (9, 7, 2, [2, 3, 31]),                          # fewer pixels than a wave; rows as long as the image
    (64, 33, 1, [2, 64, 40]),
    (70, 61, 2, [6, 141, 30]),                      # more keys in a row than one sort takes
    (40, 36, 3, [142, 12]),                         # a source grid too large for the LDS forms
    (24, 20, 4, [5 + m % 9 for m in range(66)]),    # more members than one launch takes
])
def test_members_and_adjoints(dtype, nx, ny, nsub, ns):
    import paper_1101_5803_amd as sl
    grid = sl.Grid(nx, ny, 4.0 / nx, nsub)
    G = synthgen.population(11, len(ns))
    rng = np.random.default_rng(nx)
    s = rng.standard_normal(sum(n * n for n in ns)).astype(np.float32).astype(np.float64)
    img = rng.standard_normal((len(ns), grid.J)).astype(np.float32).astype(np.float64)
    uv = sl.lens_trace(torch.tensor(G, device=DEV), grid, ns, 1.0)
    st, it = torch.tensor(s, dtype=dtype, device=DEV), torch.tensor(img, dtype=dtype, device=DEV)
    L = sl.apply_L(uv, grid, ns, st).double().cpu().numpy()
    LT = sl.apply_LT(uv, grid, ns, it).double().cpu().numpy()
    LTo = sl.apply_LT_ordered(uv, grid, ns, it)
    assert torch.equal(LTo, sl.apply_LT_ordered(uv, grid, ns, it))
    LTo = LTo.double().cpu().numpy()
    H = sl.apply_HtH("curvature", ns, st).double().cpu().numpy()
    off = 0
    for m, n in enumerate(ns):
        bx, by = olens.trace_image(G[m], nx, ny, grid.pix, nsub)
        tab = oops.bilinear_table(bx, by, n, 1.0)
        seg = slice(off, off + n * n)
        off += n * n
        if dtype == torch.float32:
            idx, w, inside = tab
            fx = (w[..., 1] + w[..., 3]).astype(np.float32).astype(np.float64)
            fy = (w[..., 2] + w[..., 3]).astype(np.float32).astype(np.float64)
            w = np.stack([(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy], axis=-1)
            tab = (idx, np.where(inside[..., None], w, 0.0), inside)
        terms = 4 * nsub * nsub
        bound = 2 * (terms + 4) * U[dtype] * oops.apply_L(tab, np.abs(s[seg]), nsub) + 1e-300
        # the traced positions agree to rounding, which moves a weight by about ns u in FP64
        bound += 64 * n * U[torch.float64] * np.abs(s[seg]).max()
        assert np.all(np.abs(L[m] - oops.apply_L(tab, s[seg], nsub)) <= bound), m
        ref = oops.apply_LT(tab, img[m], n * n, nsub)
        ones = oops.apply_LT(tab, np.abs(img[m]), n * n, nsub)
        cnt = np.bincount(np.asarray(tab[0]).reshape(-1), minlength=n * n)
        bound = 2 * (cnt + 4) * U[dtype] * ones + 64 * n * U[torch.float64] * cnt * np.abs(img[m]).max()
        assert np.all(np.abs(LT[seg] - ref) <= bound), m
        assert np.all(np.abs(LTo[seg] - ref) <= bound), m
        want = oops.apply_HtH(s[seg], n, "curvature")
        assert np.all(np.abs(H[seg] - want) <= 2 * 40 * U[dtype] * 64 * np.abs(s[seg]).max())
