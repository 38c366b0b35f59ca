"""Rows of the ordered L^T whose keys are unevenly spread: order, values and time.

The rows are built directly: subpixels of one cell at chosen places of a 256 x
256 image with 4 x 4 subpixels (4.2 M keys), everything else off the grid.
"""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
NX, NSUB = 256, 4
NSP = NX * NX * NSUB * NSUB


def _case(places):
    import paper_1101_5803_amd as sl
    uv = torch.full((1, NSP, 2), float("nan"), dtype=torch.float64)
    places = np.unique(places)
    uv[0, torch.tensor(places), 0], uv[0, torch.tensor(places), 1] = 0.25, 0.5
    img = torch.tensor(np.random.default_rng(2).standard_normal((1, NX * NX)))
    grid = sl.Grid(NX, NX, 0.01, NSUB)
    uvd, imd = uv.to(DEV), img.to(DEV)
    vals = img.numpy()[0, places // NSUB ** 2] / NSUB ** 2
    want = []
    for w in (0.75 * 0.5, 0.25 * 0.5, 0.75 * 0.5, 0.25 * 0.5):   # nodes 0, 1, ns, ns + 1; exact products
        acc = 0.0
        for v in vals:   # in key order; fma(w, v, acc) rounds once, w v is exact here but for w = 0.375
            acc = acc + w * v
        want.append(acc)
    return lambda: sl.apply_LT_ordered(uvd, grid, [3], imd), want, len(vals), np.abs(vals).sum()


def _ms(call):
    call()
    best = 1e9
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


CLUSTERS = {
    "front": [np.arange(3000), [NSP - 1]],
    "back": [[0], np.arange(NSP - 3000, NSP)],
    "middle": [[0], np.arange(NSP // 2, NSP // 2 + 3000), [NSP - 1]],
    "three": [np.arange(900), np.arange(NSP // 3, NSP // 3 + 900), np.arange(NSP - 1200, NSP)],
    "spread and dense": [np.arange(0, NSP, 4096), np.arange(5000, 7500)],
}


@pytest.mark.parametrize("name", CLUSTERS)
def test_clustered_rows(name):
    call, want, n, absum = _case(np.concatenate(CLUSTERS[name]))
    got = call()
    assert torch.equal(got, call())
    got = got.cpu().numpy()
    bound = 2 * n * 2.0 ** -53 * absum   # n fused steps here, n products and sums there
    for g, w in zip((got[0], got[1], got[3], got[4]), want):
        assert abs(g - w) <= bound
    # an evenly spread row of as many keys is scanned for ceil(n / 512) ranges; a cluster may cost the halvings down
    # to its width and the doublings back up, some tens of scans, not one per 512 keys of the whole key space
    even, _, _, _ = _case(np.linspace(0, NSP - 1, n).astype(np.int64))
    assert _ms(call) <= 8 * _ms(even) + 0.2
