"""The ordering of block lists of more than 64 entries where its method changes: by counting up to
192 (65, 191, 192 and 193 entries), by a bitmap over one and more windows of ids, by runs in LDS
beyond four windows (lists of 257 to 2048), and by merged runs (more than
24 windows and more entries than a run: 32768 ids a window and 2048 entries in the binning, 8192
and 512 in this fit).  Lists against the oracle; the fit's gradients against the standalone
calls'."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


def spread(n, K, W, H, seed):
    """K rows, of which n, spread over all ids, cover the raster; the rest lie outside it."""
    m = np.zeros((K, 7), np.float32)
    m[:, 0:2] = 1e5
    m[:, 2] = m[:, 4] = 1.0
    rng = np.random.default_rng(seed)
    at = np.unique(np.concatenate([[0, K - 1], rng.choice(K - 2, n - 2, replace=False) + 1]))
    m[at, 0], m[at, 1] = rng.uniform(0, W, n), rng.uniform(0, H, n)
    m[at, 2] = m[at, 4] = rng.uniform(30.0, 40.0, n)
    m[at, 5] = rng.normal(0.0, 0.5, n)
    m[at, 6] = rng.uniform(0, 1, n)
    return m


@pytest.mark.parametrize("scale", [1, 2])
@pytest.mark.parametrize("n,K", [(65, 65), (191, 300), (192, 70000), (193, 300), (193, 60000),
                                 (300, 120000), (193, 170000), (513, 170000), (1025, 170000),
                                 (2047, 170000), (2048, 170000), (2049, 170000), (2500, 700000),
                                 (2500, 900000), (2500, 2200000), (4100, 2200000)])
def test_lists_in_order(n, K, scale):
    import paper_2510_05814_amd as smoe
    say("sort runs", n, K, scale)
    W, H = 72, 40                     # 15 blocks: workgroups of four blocks and of three
    m_np = spread(n, K, W, H, n)
    # (a batch of that one raster: a single one takes its lists from the kernels' rectangles)
    segs = smoe.Segments([dict(width=scale * W, height=scale * H, scale=scale, num_kernels=K)])
    ob = oracle.bin(m_np, 1, 0, scale * W, scale * H, scale)
    assert int((ob["ranges"][:, 1] - ob["ranges"][:, 0]).max()) == n
    b = smoe.bin_batched(dev(m_np), 1, 0, segs, capacity=ob["P"])
    T = segs.T
    assert np.array_equal(host(b.ranges(T)), ob["ranges"])
    assert np.array_equal(host(b.vals(ob["P"])).view(np.uint32), ob["vals"])
    assert np.array_equal(host(b.keys(ob["P"])).view(np.uint32), ob["keys"])


@pytest.mark.parametrize("W,H", [(72, 40), (640, 656)])         # four waves a block, one
@pytest.mark.parametrize("n,K", [(65, 70), (192, 5000), (193, 5000), (193, 50000), (512, 50000),
                                 (513, 50000), (513, 600000), (1100, 600000)])
def test_fit_buckets_in_order(n, K, W, H):
    import torch

    import paper_2510_05814_amd as smoe
    say("sort runs, fit", n, K, W, H)
    m_np = spread(n, K, 72, 40, n)
    raw = m_np.astype(np.float64)
    raw[:, 2], raw[:, 4] = np.log(raw[:, 2]), np.log(raw[:, 4])
    t = dev(np.random.default_rng(n).uniform(0, 1, (H, W, 1)))
    T = smoe.tiles(W, H)
    st = smoe.FitState(t, dev(raw), 0, smoe.AdamConfig(total_steps=9), max_steps=1,
                       capacity=T * (n + 40))
    rows = st.model.clone()
    st.step()
    assert st.steps_done() == 1 and not st.bins.read_status()[0]
    b = smoe.bin(rows, 1, 0, smoe.make_grid(W, H))
    r, want = host(st.bins.ranges(T)), host(b.ranges(T))
    width = (T * (n + 40)) // T
    shift = int(np.ceil(np.log2(width + 16)))
    ids = host(st.bins.vals(T * width)).view(np.uint32) >> np.uint32(shift)
    vals = host(b.vals(int(want[:, 1].max()))).view(np.uint32)
    for k in range(T):
        assert np.array_equal(ids[r[k, 0]:r[k, 1]], vals[want[k, 0]:want[k, 1]]), k
    g = smoe.render_backward(rows, 1, 0, smoe.make_grid(W, H), b, st.image, st.denom, target=t)
    assert torch.equal(st.grads, g)
