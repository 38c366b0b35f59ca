"""The surrogate's kernels at the edges of their row tiles (8, 16, 32 rows) and row ranges.

Forward: a row's result is bitwise the same in a batch of any size (the rows of
a tile are independent).  Training: gradients within the bars of the gradient
test (1e-3 in norm, 1e-2 of the largest entry: BF16 roundings of activations
can flip) of the FP64 oracle.
"""
import numpy as np
import pytest
import torch

import synthgen
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _fp32(weights):
    return [(np.float32(W).astype(np.float64), np.float32(b).astype(np.float64)) for W, b in weights]


def _weights(seed):
    rng = np.random.default_rng(seed)
    return _fp32([(W, 0.1 * rng.standard_normal(b.shape)) for W, b in synthgen.mlp_init(seed)])


@pytest.mark.parametrize("batch", [7, 8, 9, 31, 2047, 2048, 2049, 4096, 4097, 20001])
def test_forward_rows_at_tile_edges(batch):
    import paper_1101_5803_amd as sl
    p = sl.mlp_pack(_weights(3), DEV)
    x = torch.tensor(synthgen.mlp_batch(5, batch)[0], dtype=torch.float32, device=DEV)
    y = sl.mlp_forward(p, x)
    rows = sorted({0, 1, 6, batch // 2, max(0, batch - 9), batch - 2, batch - 1})
    for r in rows:
        assert torch.equal(y[r:r + 1], sl.mlp_forward(p, x[r:r + 1].contiguous())), r


@pytest.mark.parametrize("batch", [1, 9, 127, 129, 257, 2049, 4097])
def test_gradients_at_tile_edges(batch):
    import paper_1101_5803_amd as sl
    w = _weights(21)
    x, yt = (np.float32(a).astype(np.float64) for a in synthgen.mlp_batch(22, batch))
    p = sl.mlp_pack(w, DEV)
    m, v, g = torch.zeros_like(p), torch.zeros_like(p), torch.full_like(p, float("nan"))
    loss = torch.empty(1, dtype=torch.float32, device=DEV)
    sl.mlp_train_step(p, m, v, torch.tensor(x, dtype=torch.float32, device=DEV),
                      torch.tensor(yt, dtype=torch.float32, device=DEV), 1e-3, 1, grads=g, loss=loss)
    lo, go = omlp.loss_and_grads(w, x, yt, quantize=True)
    assert abs(loss.item() - lo) <= 1e-4 * lo
    for (gW, gb), (oW, ob) in zip(sl.mlp_unpack(g), go):
        for got, want in ((gW, oW), (gb, ob)):
            assert np.linalg.norm(got - want) <= 1e-3 * np.linalg.norm(want)
            assert np.abs(got - want).max() <= 1e-2 * np.abs(want).max()
