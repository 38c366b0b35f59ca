"""The surrogate's forward pass allocates its output and nothing else."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


def test_forward_takes_no_workspace():
    import paper_1101_5803_amd as sl
    from paper_1101_5803_amd import ops
    B = 300_000   # its training workspace would be several hundred MB
    p = torch.zeros(sl._lib.MLP_NPARAM, device=DEV)
    p[-1] = 0.5
    x = torch.ones((B, 7), device=DEV)
    held = {k: v.numel() for k, v in ops._mlp_ws.items()}
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    y = sl.mlp_forward(p, x)
    torch.cuda.synchronize()
    assert torch.cuda.max_memory_allocated() - before <= 4 * B + (1 << 20)
    assert {k: v.numel() for k, v in ops._mlp_ws.items()} == held
    assert torch.all(y == 0.5)
    for bad in (0, sl._lib.MLP_MAX_BATCH + 1):   # refused as ever
        with pytest.raises(sl._lib.SemilinError, match="batch"):
            sl.mlp_forward(p, torch.empty((bad, 7), device=DEV))
