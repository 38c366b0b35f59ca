"""Where FP64 members of more than 94 nodes per side keep their image frame, and their results there.

A frame lies in LDS (member_info's last column) where it is sure to fit for
every member of the launch, or fits at the offsets of the launch's largest
grid; on images whose frames fit for some members only, in global memory.
Bars as in the FP64 parity tests: chi^2 1e-9, solution 1e-7, both CGs stopped
at 1e-12 and lambda >= 0.1.
"""
import ctypes

import numpy as np
import pytest
import torch

import synthgen
from oracle import mock, solve

pytestmark = pytest.mark.gpu
DEV = "cuda"
LENS = np.array([1.0, 0.75, 0.5, 0.04, 0.3, 0.02, -0.03])


def _solver(sl, n, K, R, pix, reg="identity"):
    psf = mock.gaussian_psf(K, K / 4.0)
    d = np.random.default_rng(n + K).uniform(0.0, 1.0, (n, n))
    return sl.Solver(torch.tensor(d, device=DEV), 0.1, torch.tensor(psf, device=DEV), sl.Grid(n, n, pix, 2), R, reg=reg,
                     dtype=torch.float64), d, psf


@pytest.mark.parametrize("n,K,R,theta,grids,lds", [
    (32, 5, 1.0, 1.0, [95], True),              # the only frame that this launch can have fits exactly
    (32, 5, 1.0, 1.0, [40, 95, 94], True),
    (64, 15, 1.0, 1.0, [95, 99, 100], True),    # p and a whole frame: 151 of 159 KB
    (64, 7, 1.0, 1.0, [96], True),
    (128, 5, 0.4, 0.1, [95], True),             # a small box on an image whose whole frame does not fit
    (128, 15, 1.0, 1.0, [95, 96], False),
])
def test_frames_and_results(n, K, R, theta, grids, lds):
    import paper_1101_5803_amd as sl
    pix = 4.0 / n if n < 128 else 0.05
    S, d, psf = _solver(sl, n, K, R, pix)
    lens = LENS.copy()
    lens[0] = theta
    G = np.stack([lens] * len(grids))
    ns = np.array(grids, dtype=np.int32)
    out = S.solve_semilinear(torch.tensor(G, device=DEV), torch.tensor(ns, device=DEV), (0.1, 10.0), tol=1e-12)
    info = S.member_info(int(ns.max()), len(ns), 2)
    assert np.all(info[:, 9] == int(lds)), info
    out = {k: v.cpu().numpy() for k, v in out.items()}
    for m in {0, len(grids) - 1}:
        pb = solve.Problem(G[m], d, 0.1, psf, n, n, pix, 2, int(ns[m]), R, "identity")
        assert np.all(out["status"][m] == 0)
        for k, lam in enumerate((0.1, 10.0)):
            s, _, st = solve.solve_cg(pb, lam, tol=1e-12)
            assert st == solve.ST_OK
            assert abs(out["chi2"][m, k] - pb.chi2(s)) <= 1e-9 * pb.chi2(s), (m, k)
            if k == out["k_star"][m]:
                got = out["s_corner"][out["s_off"][m]:out["s_off"][m + 1]]
                assert np.linalg.norm(got - s) <= 1e-7 * np.linalg.norm(s), (m, k)


@pytest.mark.parametrize("n,K,ns,lds", [(64, 7, 96, True), (64, 15, 99, True), (100, 5, 90, True), (128, 15, 96, False)])
def test_candidate_sources_hold_one_vector(n, K, ns, lds):
    """The candidate-source kernel keeps its frame in LDS wherever it fits beside one vector."""
    import paper_1101_5803_amd as sl
    from paper_1101_5803_amd import _lib as B
    S, d, psf = _solver(sl, n, K, 1.0, 4.0 / n)
    src = np.random.default_rng(5).uniform(0.0, 1.0, (3, ns * ns))
    got = S.chi2_sources(torch.tensor(LENS, device=DEV), ns, torch.tensor(src, device=DEV)).cpu().numpy()
    info = np.zeros((1, 10), dtype=np.int32)
    B.check(B.lib().sl_solve_member_info(ctypes.byref(S._pb), ns, 1, 1, B.ptr(S._cws),
                                         info.ctypes.data_as(ctypes.c_void_p)), "sl_solve_member_info")
    assert info[0, 9] == int(lds), info
    pb = solve.Problem(LENS, d, 0.1, psf, n, n, 4.0 / n, 2, ns, 1.0, "identity")
    for s, c in zip(src, got):
        assert abs(c - pb.chi2(s)) <= 1e-9 * c
