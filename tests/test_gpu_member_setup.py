"""The solve's member set-up (k_prep_*) at the sizes where its tiles and bands end.

Every case solves Eq. 7 with H = I at one lambda per decade and compares chi^2
and the solution with the FP64 oracle's matrix-free CG.  With both stopped at
a relative residual of 1e-12 and lambda >= 0.1 the solutions agree far below
the bars of the FP64 parity tests (chi^2 1e-9, solution 1e-7); the FP32 cases
take that path's bars (1e-5, 1e-4).  The sizes: grids of 2 nodes per side (all
pixels share four rows of the transposed operator), just below, above and at
several multiples of the 2048 nodes whose cursors one fill block holds, images
that end inside and at a 64- and 256-pixel group, fewer than 64 mapped pixels,
every subpixel count and interpolation.
"""
import numpy as np
import pytest
import torch

import synthgen
from oracle import mock, solve

pytestmark = pytest.mark.gpu
DEV = "cuda"
LAMS = (0.1, 1.0, 10.0)
CASES = [
    # nx, ny, ns, nsub, interp, dtype, half width
    (37, 33, 2, 2, "bilinear", "f64", 1.0),
    (37, 33, 2, 4, "bilinear", "f64", 1.0),
    (32, 32, 45, 2, "bilinear", "f64", 1.0),
    (32, 32, 46, 2, "bilinear", "f64", 1.0),
    (32, 24, 64, 1, "bilinear", "f64", 1.0),
    (32, 24, 91, 3, "bilinear", "f64", 1.0),
    (48, 48, 96, 2, "bilinear", "f64", 1.0),
    (9, 7, 5, 2, "bilinear", "f64", 1.0),
    (40, 36, 6, 2, "bilinear", "f64", 0.05),
    (37, 33, 46, 2, "nearest", "f64", 1.0),
    (37, 33, 12, 2, "bicubic", "f64", 1.0),
    (37, 33, 46, 4, "bicubic", "f64", 1.0),
    (37, 33, 2, 2, "bilinear", "f32", 1.0),
    (32, 32, 46, 2, "bilinear", "f32", 1.0),
    (48, 48, 91, 2, "bilinear", "f32", 1.0),
    (48, 48, 128, 2, "bilinear", "f32", 1.0),
    (37, 33, 46, 3, "bicubic", "f32", 1.0),
]


@pytest.mark.parametrize("nx,ny,ns,nsub,interp,prec,R", CASES)
def test_setup_edges_vs_oracle(nx, ny, ns, nsub, interp, prec, R):
    import paper_1101_5803_amd as sl
    pix, K = 4.0 / max(nx, ny), 5
    psf = mock.gaussian_psf(K, 1.5)
    lens = np.array([1.0, 0.75, 0.5, 0.04, 0.3, 0.02, -0.03])
    rng = np.random.default_rng(nx * 1000 + ns)
    d = rng.uniform(0.0, 1.0, (ny, nx))
    grid = sl.Grid(nx, ny, pix, nsub)
    solver = sl.Solver(torch.tensor(d, device=DEV), 0.1, torch.tensor(psf, device=DEV), grid, R, reg="identity",
                       dtype=torch.float64 if prec == "f64" else torch.float32, interp=interp)
    # a second member with another grid, so that members start inside the packed arrays
    lenses = np.stack([synthgen.population(3, 1)[0], lens])
    tol = 1e-12 if prec == "f64" else 1e-7
    grids = np.array([max(2, ns - 1), ns], dtype=np.int32)
    out = solver.solve_semilinear(torch.tensor(lenses, device=DEV), torch.tensor(grids, device=DEV), LAMS, tol=tol)
    out = {k: v.cpu().numpy() for k, v in out.items()}
    for m in range(2):
        pb = solve.Problem(lenses[m], d, 0.1, psf, nx, ny, pix, nsub, int(grids[m]), R, "identity", interp=interp)
        if np.all(out["status"][m] == sl._lib.ST_EMPTY):
            assert not np.any(pb.rhs())
            continue
        assert np.all(out["status"][m] == 0), out["status"][m]
        for k, lam in enumerate(LAMS):
            s, _, st = solve.solve_cg(pb, lam, tol=1e-12)
            assert st == solve.ST_OK
            ref = pb.chi2(s)
            assert abs(out["chi2"][m, k] - ref) <= (1e-9 if prec == "f64" else 1e-5) * ref, (m, k)
            if k == out["k_star"][m]:
                got = out["s_corner"][out["s_off"][m]:out["s_off"][m + 1]]
                err = np.linalg.norm(got - s) / np.linalg.norm(s)
                assert err <= (1e-7 if prec == "f64" else 1e-4), (m, k, err)
