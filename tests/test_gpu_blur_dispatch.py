"""Which form of the stand-alone blur a call takes, and its values on both sides of the choice.

k_blur_small runs 16 x 16 threads a block, the register-tiled forms 256 x 1.
Images that fill little of a 32 x 32 or 32 x 64 tile and PSFs too narrow for
the register window belong to the former (a register-tiled form is 1.2 to 6.5
times slower there), wide PSFs over many full tiles to the latter (1.5 to 3
times faster).  Values: as in the operators' test, within 2 (K^2 + 4) u of the
sum of absolute terms; the choice must not change a bit of an image's result.
"""
import numpy as np
import pytest
import torch

from captured import kernel_launches
from oracle import operators as oops

pytestmark = pytest.mark.gpu
DEV = "cuda"
U = {torch.float32: 2.0 ** -24, torch.float64: 2.0 ** -53}
SMALL = [(20000, 8, 8, 63), (20000, 8, 8, 3), (4096, 5, 5, 31), (65535, 4, 4, 15), (70000, 4, 4, 3), (4096, 16, 16, 63),
         (600, 200, 5, 63), (30000, 1, 33, 15), (64, 65, 65, 3), (1, 1000, 1000, 3), (1, 128, 128, 15)]
TILED = [(64, 200, 200, 21), (128, 128, 128, 15), (1, 640, 640, 63), (4096, 20, 20, 21), (16, 200, 180, 31)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,ny,nx,K,tiled", [(*c, False) for c in SMALL] + [(*c, True) for c in TILED])
def test_blur_form(dtype, n, ny, nx, K, tiled):
    import paper_1101_5803_amd as sl
    rng = np.random.default_rng(nx + K)
    P = rng.uniform(0.1, 1.0, (K, K)) / K ** 2
    x = torch.tensor(rng.standard_normal((min(n, 64), ny, nx)), device=DEV).to(torch.float32).to(dtype)
    xt = x.repeat(-(-n // len(x)), 1, 1)[:n].contiguous()
    pt = torch.tensor(P, device=DEV)
    for f, op in ((sl.apply_B, oops.apply_B), (sl.apply_BT, oops.apply_BT)):
        got = f(pt, xt)
        (_, block, _), = kernel_launches(lambda: f(pt, xt))
        assert block == ((256, 1, 1) if tiled else (16, 16, 1))
        for i in (0, n - 1):
            img = xt[i].double().cpu().numpy()
            bound = 2 * (K * K + 4) * U[dtype] * op(P, np.abs(img)) + 1e-300
            assert np.all(np.abs(got[i].double().cpu().numpy() - op(P, img)) <= bound)
            assert torch.equal(got[i], f(pt, xt[i].contiguous()))   # alone: k_blur_small, unless the image is large


def test_more_tiles_than_one_grid_dimension():
    """The register-tiled forms' grid has one dimension: past 2^31 threads the other form is taken (nothing runs here)."""
    import paper_1101_5803_amd as sl
    pt = torch.tensor(np.random.default_rng(7).uniform(0.1, 1.0, (21, 21)), device=DEV)
    sl.apply_B(pt, torch.zeros((1, 17, 17), device=DEV))
    blocks = []
    for n in (4096, 8_400_000):
        x = torch.empty((n, 17, 17), device=DEV)
        (_, block, _), = kernel_launches(lambda: sl.apply_B(pt, x))
        blocks.append(block)
        del x
    torch.cuda.empty_cache()
    assert blocks == [(256, 1, 1), (16, 16, 1)]
