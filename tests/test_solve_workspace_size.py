"""The solve's workspace holds no more per (member, lambda) than the solution and its bookkeeping."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1101_5803_amd", "libsemilin.so")


@pytest.mark.parametrize("dtype,bytes_", [("SL_F32", 4), ("SL_F64", 8)])
@pytest.mark.parametrize("n,ns", [(32, 16), (128, 64)])
def test_bytes_per_item(dtype, bytes_, n, ns):
    if not os.path.exists(LIB):
        pytest.skip("libsemilin.so not built (run python -m paper_1101_5803_amd.build)")
    from paper_1101_5803_amd import _lib as B
    size = ctypes.CDLL(LIB).sl_solve_workspace_size
    size.restype, size.argtypes = ctypes.c_size_t, [ctypes.POINTER(B.Problem)] + [ctypes.c_int] * 3
    pb = B.Problem()
    pb.img = B.ImageGrid(n, n, 0.05, 2)
    pb.sigma, pb.k, pb.half_width = 1.0, 5, 1.0
    pb.reg, pb.dtype, pb.psf_general, pb.interp = B.SL_H_CURVATURE, getattr(B, dtype), 0, 0
    M = 1000
    few, many = size(ctypes.byref(pb), ns, M, 8), size(ctypes.byref(pb), ns, M, 40)
    assert 0 < many - few <= 32 * M * (bytes_ * ns * ns + 64)


@pytest.mark.parametrize("nsub", [1, 2])
def test_bytes_per_mapped_pixel(nsub):
    """A slot of the trace table: position, the subpixels' cells and fractions, their masks, room for L^T's entries."""
    if not os.path.exists(LIB):
        pytest.skip("libsemilin.so not built (run python -m paper_1101_5803_amd.build)")
    from paper_1101_5803_amd import _lib as B
    size = ctypes.CDLL(LIB).sl_solve_workspace_size
    size.restype, size.argtypes = ctypes.c_size_t, [ctypes.POINTER(B.Problem)] + [ctypes.c_int] * 3
    pb = B.Problem()
    pb.sigma, pb.k, pb.half_width = 1.0, 5, 1.0
    pb.reg, pb.dtype, pb.psf_general, pb.interp = B.SL_H_CURVATURE, B.SL_F32, 0, 0

    def members(n, M):
        pb.img = B.ImageGrid(n, n, 0.05, nsub)
        return size(ctypes.byref(pb), 8, M, 1)
    per = [(members(n, 3001) - members(n, 1001)) / 2000 for n in (128, 256)]   # the per-block scratch cancels
    slot = (per[1] - per[0]) / (256 * 256 - 128 * 128)
    assert slot <= 4 + 12 * nsub ** 2 + 64 * nsub ** 2 + 2.01
