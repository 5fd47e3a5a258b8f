"""Binning of batches by native block (scales of 2 to 8, and with a scale of 9 among them, whose
scale^2 output blocks of a native block share their list): rasters that begin and
end inside a native block on either side of zero, scale-1 rasters beside them, lists of up to 64
entries and of hundreds, rasters without kernels, and an overflow.  Every raster's arrays against
the oracle's."""
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


#          width, height, scale, origin_x, origin_y, kernels
RASTERS = [(150, 90, 2, 0, 0, 60), (70, 33, 1, 0, 0, 40), (333, 211, 3, 7, -50, 50),
           (65, 65, 4, 0, 0, 0), (190, 260, 4, -37, 91, 90), (129, 300, 8, 120, -129, 70),
           (16, 16, 8, 16, 112, 5), (40, 20, 1, -8, 5, 30)]


@pytest.mark.parametrize("nine", [False, True])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("trunc", ["gradient", "render"])
def test_lists_against_oracle(smoe, trunc, wide, nine):
    say("shared lists", trunc, wide, nine)
    rasters = RASTERS + ([(100, 50, 9, 3, 0, 20)] if nine else [])
    if wide:
        rasters = [r[:5] + (r[5] * 5,) for r in rasters]
    models = [wl.random_model(K, 1, 0, -(-W // s), -(-H // s), K + W, sig_lo=1.0,
                              sig_hi=30.0 if wide else 3.0) for W, H, s, _, _, K in rasters]
    segs = smoe.Segments([dict(width=W, height=H, scale=s, origin_x=ox, origin_y=oy,
                               num_kernels=K) for W, H, s, ox, oy, K in rasters])
    m = dev(np.concatenate(models))
    want = [oracle.bin(mm, 1, 0, W, H, s, ox, oy, trunc=trunc)
            for mm, (W, H, s, ox, oy, _) in zip(models, rasters)]
    P = sum(o["P"] for o in want)
    b = smoe.Bins(segs.K, 1, 0, segs.T, P, render_only=True)
    for fill in (0xFF, 0x00):
        b.ws.fill_(fill)
        smoe.bin_batched(m, 1, 0, segs, bins=b, grow=False, trunc=trunc)
        over, st = b.read_status()
        longest = max(int((o["ranges"][:, 1] - o["ranges"][:, 0]).max()) for o in want)
        assert not over and st[0] == P and st[2] == longest and (longest > 64) == wide
        ranges, keys = host(b.ranges(segs.T)), host(b.keys(P)).view(np.uint32)
        vals = host(b.vals(P)).view(np.uint32)
        at = 0
        for o, sg in zip(want, segs.host):
            T, t0, k0, K = len(o["ranges"]), sg.tile_offset, sg.kernel_offset, sg.num_kernels
            p = o["P"]
            assert np.array_equal(ranges[t0:t0 + T, 1] - ranges[t0:t0 + T, 0],
                                  o["ranges"][:, 1] - o["ranges"][:, 0])
            assert np.array_equal(vals[at:at + p], o["vals"] + np.uint32(k0))
            assert np.array_equal(keys[at:at + p], o["keys"] + np.uint32(t0))
            assert np.array_equal(host(b.counts())[k0:k0 + K], o["counts"])
            assert np.array_equal(host(b.tile_rects())[k0:k0 + K], o["tile_rects"])
            at += p
        assert not host(b._view(b.c.tile_counts, segs.T, ranges_dtype())).any()
    small = smoe.Bins(segs.K, 1, 0, segs.T, P - 1, render_only=True)
    smoe.bin_batched(m, 1, 0, segs, bins=small, grow=False, trunc=trunc)
    over, st = small.read_status()
    assert over and st[0] == P and not host(small.ranges(segs.T)).any()


def ranges_dtype():
    import torch
    return torch.int32
