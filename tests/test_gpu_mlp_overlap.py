"""GPU: lbw_mlp_forward on inputs and outputs that share memory gives the bits
of separate buffers: y over x from its start, behind and before it, with wider
and narrower outputs, and in place; rows enough for many workgroups.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw
from oracle import mlp as ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [[3, 40, 10], [10, 40, 3], [6, 32, 6], [9, 2], [3, 300, 10]], ids=str)
@pytest.mark.parametrize("B", [5, 4097])
def test_outputs_over_inputs(widths, B):
    print("mlp overlap", widths, B, flush=True)
    rng = np.random.default_rng(B)
    net = lbw.MLP(widths, max_batch=B)
    net.set_params(ref.init_params(widths, rng))
    x = torch.as_tensor(rng.uniform(-1, 1, size=(B, widths[0])).astype(np.float32), device="cuda")
    y = net.forward(x)
    nx, ny = x.numel(), y.numel()
    for x_at, y_at in ((0, 0), (0, nx // 2), (ny // 2, 0), (0, nx - 1), (ny - 1, 0), (0, nx), (ny, 0)):
        buf = torch.full((nx + ny,), 7.0, dtype=torch.float32, device="cuda")
        buf[x_at:x_at + nx] = x.reshape(-1)
        lbw.check(lbw.lib().lbw_mlp_forward(net.handle, buf[x_at:].data_ptr(), B, buf[y_at:].data_ptr()))
        assert torch.equal(buf[y_at:y_at + ny].reshape(B, -1), y), (x_at, y_at)
    assert torch.equal(net.forward(x), y)
