"""Batches of more rasters than the table is bisected for (64): the search by interpolation over
uneven rasters -- single blocks, large ones in between, models without kernels, runs of equal
offsets -- finds every kernel's and every block's raster.  Lists against the oracle's, raster
by raster."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kind", [(64, "uneven"), (65, "uneven"), (300, "uneven"), (200, "windows"),
                                    (130, "empty")])
def test_lists_of_many_segments(n, kind):
    import paper_2510_05814_amd as smoe
    say("segments", n, kind)
    rng = np.random.default_rng(n)
    rasters, models, base = [], [], 0
    for i in range(n):
        side = 16 if kind == "windows" else int(rng.choice([5, 16, 33, 200 if i % 40 == 7 else 20]))
        K = 4 if kind == "windows" else int(rng.choice([0, 1, 3, 90 if i % 40 == 7 else 6]))
        if kind == "empty" and i not in (0, 70, 129):
            K = 0
        models.append(wl.random_model(K, 1, 0, side, side, i).astype(np.float32))
        rasters.append(dict(width=side, height=side, num_kernels=K, param_offset=base))
        base += K
    params = np.concatenate(models)
    segs = smoe.Segments(rasters)
    b = smoe.bin_batched(dev(params), 1, 0, segs)
    P = b.read_status()[1][0]
    vals, ranges = host(b.vals(P)).view(np.uint32), host(b.ranges(segs.T))
    rects = host(b.tile_rects())
    p0 = 0
    for sg, m, r in zip(segs.host, models, rasters):
        o = oracle.bin(m, 1, 0, r["width"], r["height"])
        k0, t0, T = sg.kernel_offset, sg.tile_offset, len(o["ranges"])
        assert np.array_equal(rects[k0:k0 + len(m)], o["tile_rects"])
        assert np.array_equal(ranges[t0:t0 + T], o["ranges"] + p0)
        assert np.array_equal(vals[p0:p0 + o["P"]], o["vals"] + k0)
        p0 += o["P"]
    assert p0 == P
