"""The scan of the block counts of a large raster whose pair storage has no room for the chunks'
sums: each workgroup walks several chunks of 4096 blocks, the last workgroup fewer and the last
chunk part of one.  Lists against the oracle's, whole, and an overflow."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


#                                blocks: 17, 33 and 65 chunks by 9, 11 and 13 workgroups
@pytest.mark.parametrize("W,H", [(4112, 4112), (8192, 4100), (8200, 8200)])
def test_ranges_against_oracle(W, H):
    import paper_2510_05814_amd as smoe
    say("scan, few pairs", W, H)
    K = 9
    rng = np.random.default_rng(W)
    m_np = np.zeros((K, 7), np.float32)
    m_np[:, 0], m_np[:, 1] = rng.uniform(0, W, K), rng.uniform(0, H, K)
    m_np[:, 2:5] = [3.0, 0.5, 4.0]
    m_np[:4, 0:2] = [[1.0, 1.0], [W - 1.0, H - 1.0], [W - 1.0, 1.0], [W / 2, H - 30.0]]
    grid = smoe.make_grid(W, H)
    ob = oracle.bin(m_np, 1, 0, W, H)
    T, P = smoe.tiles(W, H), ob["P"]
    assert P // 4 < -(-T // 4096)
    for capacity in (P, P - 1):
        b = smoe.Bins(K, 1, 0, T, capacity, render_only=True)
        b.ws.fill_(0xFF)
        smoe.bin(dev(m_np), 1, 0, grid, bins=b, grow=False)
        over, st = b.read_status()
        assert over == (capacity < P) and st[0] == P
        assert st[2] == int((ob["ranges"][:, 1] - ob["ranges"][:, 0]).max())
        r = host(b.ranges(T))
        n = r[:, 1] - r[:, 0]
        if over:
            assert not r.any()
            continue
        assert np.array_equal(n, ob["ranges"][:, 1] - ob["ranges"][:, 0])
        assert np.array_equal(r[n > 0], ob["ranges"][n > 0])
        assert np.array_equal(host(b.vals(P)).view(np.uint32), ob["vals"])
        assert np.array_equal(host(b.keys(P)).view(np.uint32), ob["keys"])
