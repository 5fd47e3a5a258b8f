"""The scan of block counts where it changes: rasters of one and of several chunks of 4096 blocks,
with a partial last chunk, of more than 65536 blocks (the chunks' sums from a launch of their
own), with too little pair storage for those sums, and an overflow over several chunks.  Lists
against the oracle's, whole."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


#                 W, H: 4096, 4097 + ..., 8192 + ... and 66049 blocks
@pytest.mark.parametrize("W,H,K,capacity", [(1024, 1024, 60, None), (1040, 1024, 60, None),
                                            (2048, 1041, 90, None), (4112, 4112, 40, None),
                                            (4112, 4112, 3, 60)])
def test_ranges_against_oracle(smoe, W, H, K, capacity):
    say("scan", W, H, K, capacity)
    rng = np.random.default_rng(K)
    m_np = np.zeros((K, 7), np.float32)
    m_np[:, 0], m_np[:, 1] = rng.uniform(0, W, K), rng.uniform(0, H, K)
    m_np[:, 2:5] = [3.0, 0.5, 4.0]
    m_np[:3, 0:2] = [[1.0, 1.0], [W - 1.0, H - 1.0], [W - 1.0, 1.0]]   # the corners' blocks
    grid = smoe.make_grid(W, H)
    ob = oracle.bin(m_np, 1, 0, W, H)
    T = smoe.tiles(W, H)
    b = smoe.Bins(K, 1, 0, T, capacity or ob["P"], render_only=True)
    b.ws.fill_(0xFF)
    smoe.bin(dev(m_np), 1, 0, grid, bins=b, grow=False)
    over, st = b.read_status()
    assert not over and st[0] == ob["P"] and st[2] == int((ob["ranges"][:, 1] - ob["ranges"][:, 0]).max())
    r = host(b.ranges(T))
    n = r[:, 1] - r[:, 0]
    assert np.array_equal(r[n > 0], ob["ranges"][n > 0]) and np.array_equal(n, ob["ranges"][:, 1] - ob["ranges"][:, 0])
    assert np.array_equal(host(b.vals(ob["P"])).view(np.uint32), ob["vals"])
    assert np.array_equal(host(b.keys(ob["P"])).view(np.uint32), ob["keys"])
    # an overflow empties every range and the next binning is whole again
    small = smoe.Bins(K, 1, 0, T, ob["P"] - 1, render_only=True)
    smoe.bin(dev(m_np), 1, 0, grid, bins=small, grow=False)
    over, st = small.read_status()
    assert over and st[0] == ob["P"] and not host(small.ranges(T)).any()
