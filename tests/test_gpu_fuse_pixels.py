"""Window fusion straight from the windows (a thread per pixel) where its loads ahead change -- 1, 2,
3, 4, 5, 8 and 9 windows an axis, 32 of them -- and on both sides of the rule that sends a call by
way of LDS instead: window and displacement, and window renders just over 256 MiB.  Against the
sum over the covering windows in (window row, window column) order on the host, bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_fuse_windows import spans
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


#                          W, H, window, displacement
@pytest.mark.parametrize("W,H,w,d", [
    (67, 9, 5, 5), (130, 37, 14, 7), (65, 33, 33, 11), (64, 40, 36, 9), (100, 21, 55, 11),
    (71, 30, 24, 3), (66, 29, 27, 3), (129, 20, 64, 2), (70, 19, 32, 2), (70, 19, 34, 2),
    (50, 18, 3, 1), (50, 18, 4, 1), (90, 17, 6, 2), (90, 17, 8, 2), (1, 300, 1024, 4),
    (1210, 1160, 16, 4)])
@pytest.mark.parametrize("C", [1, 3])
def test_sum_in_window_order(W, H, w, d, C):
    import paper_2510_05814_amd as smoe
    say("fuse pixels", W, H, w, d, C)
    m = w // d
    rng = np.random.default_rng(W + 5 * w + C)
    win = rng.standard_normal((m * m * W * H, C), dtype=np.float32)
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
