"""The differentiable render of a model whose pairs exceed the workspace it starts with: it renders
again with a larger one.  Image and gradient are those of the calls it is made of, with room from
the start, bit for bit."""
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,K,order", [(160, 150, 200, 1), (1300, 1290, 90, 0)])
def test_image_and_gradient(W, H, K, order):
    import torch

    import paper_2510_05814_amd as smoe
    from paper_2510_05814_amd.autograd import smoe_render
    say("autograd overflow", W, H, K)
    m = dev(wl.random_model(K, 3, order, W, H, K, sig_lo=0.15 * W, sig_hi=0.3 * W))
    raw = m.clone()
    raw[:, 2], raw[:, 4] = raw[:, 2].log(), raw[:, 4].log()
    raw.requires_grad_(True)
    up = dev(wl.random_model(H * W, 1, 0, W, H, 4)[:, 4:7].reshape(H, W, 3))
    img = smoe_render(raw, 3, order, W, H)
    img.backward(up)
    rows = smoe.materialize(raw.detach(), 3, order)
    grid = smoe.make_grid(W, H, trunc="render")
    T = smoe.tiles(W, H)
    b = smoe.bin(rows, 3, order, grid, capacity=K * T)
    P = b.read_status()[1][0]
    assert P > smoe.core.initial_capacity(K, T)       # the first workspace is too small
    want, D, _, _ = smoe.render(rows, 3, order, grid, bins=b)
    g = smoe.render_backward(rows, 3, order, grid, b, want, D, grad_image=up)
    assert torch.equal(img.detach(), want) and torch.equal(raw.grad, g)
