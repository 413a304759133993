"""GPU: the few-launch path of small networks at the sizes where it changes:
layer widths around 16-column tiles and 32-term steps, one and eight layers
(nine, and a layer of 257 units, take the general path), batches on both
sides of each number of rows per workgroup (4, 8, 16 .. 64 times 256 CUs), and
of one row.

Bars as in the surrogate kernels' other tests, and for the same reason
(isolated BF16 rounding flips between FP32 on the device and FP64 on the
host, 2^-8 of one activation each): relative L2 2e-4 for outputs, 1e-3 for
gradients, 1e-4 for the loss; networks of one layer have no activation to flip
and are held to 1e-5.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw
from oracle import mlp as ref

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(b))


@pytest.mark.parametrize("widths", [[1, 1], [256, 256], [3, 15, 10], [3, 16, 17, 1], [31, 32, 33, 5],
                                    [64, 65, 128, 129, 2], [7, 255, 256, 3], [3] + [24] * 7 + [4],
                                    [3] + [24] * 8 + [4], [3, 257, 2]], ids=str)
@pytest.mark.parametrize("B", [1, 33])
def test_few_layers_match_reference(widths, B):
    print("mlp few", widths, B, flush=True)
    rng = np.random.default_rng(len(widths) * 1000 + B)
    p = ref.init_params(widths, rng)
    p = (p + rng.normal(scale=0.02, size=p.size)).astype(np.float32).astype(np.float64)
    x = rng.uniform(-1, 1, size=(B, widths[0])).astype(np.float32).astype(np.float64)
    t = rng.normal(size=(B, widths[-1])).astype(np.float32).astype(np.float64)
    w = rng.uniform(0.5, 1.5, size=(B, widths[-1])).astype(np.float32).astype(np.float64)
    net = lbw.MLP(widths, max_batch=40)
    net.set_params(p)
    bar = (1e-5, 1e-5) if len(widths) == 2 else (2e-4, 1e-3)
    yr, _ = ref.forward(p, widths, x)
    assert rel(net.forward(x).cpu().numpy(), yr) <= bar[0]
    loss, grad = net.loss_grad(x, t, w, want_grad=True)
    lr_, gr = ref.loss_grad(p, widths, x, t, w)
    assert abs(loss.item() - lr_) <= 1e-4 * abs(lr_)
    assert rel(grad.cpu().numpy(), gr) <= bar[1]


@pytest.mark.parametrize("B", [1024, 1025, 2049, 4097, 8193, 12289])
def test_rows_do_not_depend_on_the_batch(B):
    """Every row comes out the same whatever the number of rows that share
    its workgroup, and a training step's gradient is that of a batch split in
    two (FP32 sums: 1e-5)."""
    print("mlp rows", B, flush=True)
    widths = [3, 40, 17, 10]
    rng = np.random.default_rng(B)
    p = ref.init_params(widths, rng)
    net = lbw.MLP(widths, max_batch=B)
    net.set_params(p)
    x = torch.as_tensor(rng.uniform(-1, 1, size=(B, 3)).astype(np.float32), device="cuda")
    t = torch.as_tensor(rng.normal(size=(B, 10)).astype(np.float32), device="cuda")
    y = net.forward(x)
    for a, b in ((0, 1), (B // 2 - 3, B // 2 + 700), (B - 5, B)):
        assert torch.equal(net.forward(x[a:b]), y[a:b])
    _, g = net.loss_grad(x, t, want_grad=True, weight_sum=10.0 * B)
    parts = [net.loss_grad(x[s], t[s], want_grad=True, weight_sum=10.0 * B)[1].double()
             for s in (slice(0, B // 3), slice(B // 3, B))]
    assert rel(g.double().cpu().numpy(), (parts[0] + parts[1]).cpu().numpy()) <= 1e-5
