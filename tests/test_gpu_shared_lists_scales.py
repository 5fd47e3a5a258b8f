"""Lists shared by native block at large scales (9 to 64, where a native block has 81 to 4096
output blocks): rasters inside one native block, across several, with origins inside one on either
side of zero.  Every raster's lists against the oracle's."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu

#          width, height, scale, origin_x, origin_y, kernels
RASTERS = [(300, 170, 9, 100, -200, 30), (500, 260, 16, -130, 77, 40), (90, 1500, 33, 500, -700, 35),
           (2100, 70, 64, -1000, 900, 50), (40, 33, 64, 1030, -1023, 12), (33, 50, 1, -7, 0, 20)]


@pytest.mark.parametrize("wide", [False, True])
def test_lists_against_oracle(wide):
    import paper_2510_05814_amd as smoe
    say("shared lists, large scales", wide)
    rasters = [r[:5] + (r[5] * 7,) for r in RASTERS] if wide else RASTERS
    models = []
    for i, (W, H, s, ox, oy, K) in enumerate(rasters):
        m = wl.random_model(K, 1, 0, W // s + 1, H // s + 1, i, sig_lo=1.0,
                            sig_hi=30.0 if wide else 5.0)
        m[:, 0] += ox / s
        m[:, 1] += oy / s
        models.append(m)
    segs = smoe.Segments([dict(width=W, height=H, scale=s, origin_x=ox, origin_y=oy, num_kernels=K)
                          for W, H, s, ox, oy, K in rasters])
    want = [oracle.bin(m, 1, 0, W, H, s, ox, oy)
            for m, (W, H, s, ox, oy, _) in zip(models, rasters)]
    P = sum(o["P"] for o in want)
    b = smoe.bin_batched(dev(np.concatenate(models)), 1, 0, segs, capacity=P)
    over, st = b.read_status()
    longest = max(int((o["ranges"][:, 1] - o["ranges"][:, 0]).max()) for o in want)
    assert not over and st[0] == P and st[2] == longest and (longest > 192) == wide
    ranges, keys = host(b.ranges(segs.T)), host(b.keys(P)).view(np.uint32)
    vals = host(b.vals(P)).view(np.uint32)
    at = 0
    for o, sg in zip(want, segs.host):
        T, t0, p = len(o["ranges"]), sg.tile_offset, o["P"]
        assert np.array_equal(ranges[t0:t0 + T, 1] - ranges[t0:t0 + T, 0],
                              o["ranges"][:, 1] - o["ranges"][:, 0])
        assert np.array_equal(vals[at:at + p], o["vals"] + np.uint32(sg.kernel_offset))
        assert np.array_equal(keys[at:at + p], o["keys"] + np.uint32(t0))
        at += p
