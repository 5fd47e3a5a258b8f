"""Block lists read off the kernels' rectangles (small single rasters) against the counted and
sorted ones (a batch of that one raster takes the general path): every array the binning leaves,
word for word, at the edges of the rule -- one workgroup or several, a partial last one, a chunk of
64 kernels or 256, 4096 blocks and 4097 -- with odd sizes, windows, scales, sharpening, both boxes
and truncations, rows that take no part, and an overflow."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


CASES = [
    # W, H, K, grid options; blocks
    (16, 16, 1, {}),                                               # 1
    (64, 64, 64, {}),                                              # 16
    (512, 32, 64, {}),                                             # 64: the largest at once
    (1040, 16, 64, {}),                                            # 65: several workgroups
    (32, 64, 512, {"box": "tight"}),                               # 8 and 8 chunks
    (32, 64, 513, {"box": "tight"}),                               # 8 and 9 chunks
    (125, 127, 513, {"trunc": "render"}),                          # 64
    (512, 256, 64, {}),                                            # 512
    (513, 256, 64, {}),                                            # 528
    (8192, 16, 60, {"origin_x": 7}),                               # 513
    (509, 381, 3024, {"trunc": "render"}),                         # 768
    (512, 512, 4096, {"scale": 2, "origin_x": 5, "origin_y": -7}),
    (301, 203, 700, {"scale": 3, "sharpen": 1.5}),
    (97, 211, 900, {"scale": 4, "origin_x": -33, "box": "tight"}),
    (32, 32, 16384, {}),                                           # 4 blocks, 256 chunks
    (32, 32, 16385, {}),                                           # the general path twice
    (1024, 1024, 8192, {}),                                        # 4096 blocks, 2^25 pairs
    (1024, 1024, 8193, {}),                                        # the general path twice
    (1040, 1024, 1000, {}),                                        # 4160: the general path twice
]


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("W,H,K,opts", CASES)
def test_same_as_counted_and_sorted(smoe, W, H, K, opts, wide):
    import torch
    say("block lists", W, H, K, opts, wide)
    if wide and K * W * H > 2 ** 31:
        K //= 16
    opts = dict(opts)
    s = opts.get("scale", 1)
    m_np = wl.random_model(K, 1, 0, -(-W // s), -(-H // s), K + W, sig_lo=1.0,
                           sig_hi=60.0 if wide else 4.0)
    m_np[K // 3, 0], m_np[K // 2, 2] = 1e6, 1e-6           # outside the raster; no pixel centre
    if wide:
        m_np[K // 5, 3], m_np[K - 1, 6] = np.nan, np.inf
    m = dev(m_np)
    segs = smoe.Segments([dict(width=W, height=H, num_kernels=K,
                               **{k: v for k, v in opts.items()
                                  if k in ("scale", "origin_x", "origin_y", "sharpen")})])
    how = {k: v for k, v in opts.items() if k in ("box", "trunc")}
    want = smoe.bin_batched(m, 1, 0, segs, **how)
    P, T = want.read_status()[1][0], segs.T
    got = smoe.Bins(K, 1, 0, T, max(P, 1), render_only=True)
    for fill in (0xFF, 0x00):
        got.ws.fill_(fill)
        smoe.bin(m, 1, 0, smoe.make_grid(W, H, **opts), bins=got, grow=False)
        over, st = got.read_status()
        assert not over and st == want.read_status()[1]
        for name, arg in (("tile_rects", ()), ("native_rects", ()), ("counts", ()),
                          ("ranges", (T,)), ("keys", (P,)), ("vals", (P,))):
            assert torch.equal(getattr(got, name)(*arg), getattr(want, name)(*arg)), name
        n = K * got.c.record_stride
        assert torch.equal(got._view(got.c.records, n, torch.int32),
                           want._view(want.c.records, n, torch.int32))
        assert not got._view(got.c.tile_counts, T, torch.int32).any()
    if P > 1:
        small = smoe.Bins(K, 1, 0, T, P - 1, render_only=True)
        small.ws.fill_(0xFF)
        smoe.bin(m, 1, 0, smoe.make_grid(W, H, **opts), bins=small, grow=False)
        over, st = small.read_status()
        assert over and st[0] == P and st[2] == want.read_status()[1][2]
        assert not host(small.ranges(T)).any()
        assert (small.vals(P - 1) == -1).all()
