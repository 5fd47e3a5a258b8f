"""The ordering of long block lists by a bitmap of the ids present: lists of 64, 65 and more ids,
ids spread over one and several windows of the bitmap (32768 ids in the binning, 8192 in the
fit step), on their edges, and several long lists in the same workgroup beside short ones.
Lists against the oracle; a fit whose buckets hold them against the standalone calls, bit for
bit."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


def spread(n, K, gap_first, W, H, seed):
    """K rows, of which n, `gap_first` ids apart, cover the raster; the rest lie outside it."""
    m = wl.random_model(K, 1, 0, W, H, seed, sig_lo=1.0, sig_hi=3.0).astype(np.float64)
    m[:, 0] += 1e5
    at = (np.arange(n) * gap_first) % K
    at[-1] = K - 1
    at = np.unique(at)
    rng = np.random.default_rng(seed)
    m[at, 0] = rng.uniform(0, W, len(at))
    m[at, 1] = rng.uniform(0, H, len(at))
    m[at, 2] = m[at, 4] = rng.uniform(8.0, 20.0, len(at))
    m[at, 3] = 0.0
    return m.astype(np.float32)


@pytest.mark.parametrize("n,K,gap", [(64, 64, 1), (65, 65, 1), (130, 400, 3), (300, 8193, 27),
                                     (90, 32769, 364), (700, 70000, 100), (200, 66000, 8192)])
def test_long_lists_in_order(smoe, n, K, gap):
    import torch
    say("sort lists", n, K, gap)
    W, H = 72, 40                     # 15 blocks: workgroups of four blocks and of three
    m_np = spread(n, K, gap, W, H, 7 + n)
    m, grid = dev(m_np), smoe.make_grid(W, H)
    b = smoe.bin(m, 1, 0, grid)
    ob = oracle.bin(m_np, 1, 0, W, H)
    assert np.array_equal(host(b.ranges(15)), ob["ranges"])
    assert np.array_equal(host(b.vals(ob["P"])).view(np.uint32), ob["vals"])
    assert np.array_equal(host(b.keys(ob["P"])).view(np.uint32), ob["keys"])
    raw = m_np.astype(np.float64)
    raw[:, 2], raw[:, 4] = np.log(raw[:, 2]), np.log(raw[:, 4])
    t = dev(np.random.default_rng(n).uniform(0, 1, (H, W, 1)))
    longest = int((ob["ranges"][:, 1] - ob["ranges"][:, 0]).max())
    st = smoe.FitState(t, dev(raw), 0, smoe.AdamConfig(total_steps=9), max_steps=1,
                       capacity=15 * (longest + 40))
    rows = st.model.clone()
    img, D, _, b = smoe.render(rows, 1, 0, grid)
    st.step()
    assert st.steps_done() == 1 and not st.bins.read_status()[0]
    if longest <= 128:                # (longer lists: the render sums quarters)
        assert torch.equal(st.image, img) and torch.equal(st.denom, D)
    want = smoe.render_backward(rows, 1, 0, grid, b, st.image, st.denom, target=t)
    assert torch.equal(st.grads, want)
