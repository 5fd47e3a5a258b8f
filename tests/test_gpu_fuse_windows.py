"""Window fusion where a wave's copies change: windows of 1 to 1024 pixels (one lane a window to
whole waves of them), rows of windows that fit one batch and several, window sizes that are no
power of two, images narrower than a window, a last tile of one pixel.  Against the sum over
the covering windows in (window row, window column) order on the host, bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


def spans(n, d, w):
    k = np.arange(-(-n // d) + w // d - 1)
    return np.maximum(0, (k + 1) * d - w), np.minimum(n, (k + 1) * d)


#                          W, H, window, displacement
@pytest.mark.parametrize("W,H,w,d", [
    (1, 1, 16, 2), (65, 9, 16, 2), (130, 70, 16, 1), (64, 5, 16, 16), (67, 33, 16, 8),
    (129, 6, 1, 1), (66, 7, 3, 1), (100, 50, 24, 8), (70, 21, 33, 11), (200, 40, 64, 16),
    (130, 131, 65, 13), (90, 20, 1024, 256), (1100, 3, 1024, 512), (5, 300, 128, 64)])
@pytest.mark.parametrize("C", [1, 3])
def test_sum_in_window_order(W, H, w, d, C):
    import torch

    import paper_2510_05814_amd as smoe
    say("fuse", W, H, w, d, C)
    m = w // d
    rng = np.random.default_rng(W + 7 * w + C)
    win = rng.standard_normal((m * m * W * H, C)).astype(np.float32)
    ax, bx = spans(W, d, w)
    ay, by = spans(H, d, w)
    acc = np.zeros((H, W, C), np.float32)
    at = 0
    for y0, y1 in zip(ay, by):
        for x0, x1 in zip(ax, bx):
            n = (y1 - y0) * (x1 - x0)
            acc[y0:y1, x0:x1] += win[at:at + n].reshape(y1 - y0, x1 - x0, C)
            at += n
    assert at == m * m * W * H
    want = acc / np.float32(m * m)
    got = host(smoe.fuse_windows(dev(win), C, W, H, d, w))
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
