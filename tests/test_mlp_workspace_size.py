"""A workspace sized for a program's largest minibatch holds every smaller one.

sl_mlp_train_step takes no workspace size, so the size must not fall where the
rows per block change (2048 and 4096 rows) or anywhere else.
"""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1101_5803_amd", "libsemilin.so")


def test_size_never_falls_with_the_batch():
    if not os.path.exists(LIB):
        pytest.skip("libsemilin.so not built (run python -m paper_1101_5803_amd.build)")
    size = ctypes.CDLL(LIB).sl_mlp_workspace_size
    size.restype, size.argtypes = ctypes.c_size_t, [ctypes.c_int]
    batches = list(range(0, 10000)) + list(range(10000, 1 << 20, 997)) + [(1 << 20) - 1, 1 << 20]
    sizes = [size(b) for b in batches]
    assert sizes[0] > 0
    falls = [(b, s, t) for b, s, t in zip(batches, sizes, sizes[1:]) if t < s]
    assert not falls, falls[:5]
