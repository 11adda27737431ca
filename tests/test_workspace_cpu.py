"""Workspace sizes that programs have allocated once and keep: what a size was
enough for stays enough."""
import numpy as np
import pytest
import torch

from paper_2207_00426_amd import pss


@pytest.mark.parametrize("B,n,size", [(64, 10000, 456957696), (8, 1500, 8638976),
                                      (1, 5000, 3573504), (300, 600, 127869952)])
def test_fp32_gradient_needs_no_more_than_its_tiled_adjoint_scan(B, n, size):
    b = pss.Batch(pss.MODEL_CT, torch.float32, 5, 2, np.arange(B + 1) * n, np.zeros(5), np.eye(5),
                  device="cpu", dt=0.01)
    assert pss.workspace_size(b, "loglik_grad") <= size
