"""GPU: the forward pass of batches of more rows than one round of workgroups
takes, in workgroups of four, eight and sixteen waves: widths on both sides of
64 and 128 units, inputs on both sides of 64, one layer and several.  Every row
is the same bits as in a small batch (which other tests hold to the reference).
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw
from oracle import mlp as ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [[1, 1], [64, 64], [65, 3], [3, 64, 64, 10], [3, 65, 10], [64, 65, 64], [128, 128],
                                    [8, 128], [70, 128, 65, 2], [129, 8], [3, 129, 10], [3] + [40] * 7 + [10]], ids=str)
@pytest.mark.parametrize("B", [12288, 12289, 16385, 50001])
def test_rows_of_large_batches(widths, B):
    print("mlp many rows", widths, B, flush=True)
    rng = np.random.default_rng(B)
    net = lbw.MLP(widths, max_batch=B)
    net.set_params(ref.init_params(widths, rng))
    x = torch.as_tensor(rng.uniform(-1, 1, size=(B, widths[0])).astype(np.float32), device="cuda")
    y = net.forward(x)
    for a, b in ((0, 1), (60, 200), (B // 2 - 3, B // 2 + 700), (B - 70, B)):
        assert torch.equal(net.forward(x[a:b]), y[a:b]), (a, b)
