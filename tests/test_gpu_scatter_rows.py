"""The binning's appends with four lanes a kernel row, whose blocks past the sixteenth the lanes of four
rows take together: rows of no block, of 12, 16, 20, 80, 81 and of hundreds side by side, a last group
of one to three rows; single rasters of many kernels, at scale 1 and (lists shared by native block)
3, and batches of small rasters with a large one among them.  Lists against the oracle's."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu

SIZES = [(9.0, 9.0), (10.5, 10.5), (14.0, 24.0), (40.0, 2.0), (2.0, 60.0), (45.0, 45.0),
         (0.01, 0.01)]


def rows(K, W, H, seed):
    """Narrow kernels, every 37th with a box of one of the SIZES, some outside the raster."""
    m = wl.random_model(K, 1, 0, W, H, seed, sig_lo=0.5, sig_hi=1.5, margin=20.0)
    for k in range(0, K, 37):
        m[k, 2], m[k, 4] = SIZES[k // 37 % len(SIZES)]
        m[k, 3] = 0.0
    m[-1, 0:5] = [W / 2, H / 2, 50.0, 3.0, 40.0]
    return m


def check(b, T, ob, t0=0, k0=0, at=0):
    P = ob["P"]
    r = host(b.ranges(t0 + T))[t0:]
    assert np.array_equal(r[:, 1] - r[:, 0], ob["ranges"][:, 1] - ob["ranges"][:, 0])
    assert np.array_equal(host(b.vals(at + P))[at:].view(np.uint32), ob["vals"] + np.uint32(k0))
    assert np.array_equal(host(b.keys(at + P))[at:].view(np.uint32), ob["keys"] + np.uint32(t0))
    return at + P


@pytest.mark.parametrize("K", [16385, 16386, 16387, 20001])
@pytest.mark.parametrize("s,ox", [(1, 0), (3, 7)])
def test_many_kernels(K, s, ox):
    import paper_2510_05814_amd as smoe
    say("scatter rows", K, s)
    W, H = 400, 333
    m_np = rows(K, W, H, K + s)
    ob = oracle.bin(m_np, 1, 0, s * W, s * H, s, ox, -ox)
    assert ob["counts"].max() > 200
    assert s > 1 or {0, 1, 12, 16, 20, 80, 81} < set(ob["counts"].tolist())
    b = smoe.bin(dev(m_np), 1, 0, smoe.make_grid(s * W, s * H, s, ox, -ox), capacity=ob["P"])
    over, st = b.read_status()
    assert not over and st[0] == ob["P"]
    check(b, len(ob["ranges"]), ob)


def test_small_rasters_and_a_large_one():
    import paper_2510_05814_amd as smoe
    say("scatter rows, batch")
    rasters = [(16 + i % 3, 20, 3 + i % 4) for i in range(60)] + [(300, 260, 149)] + [(17, 16, 2)] * 20
    models = [rows(K, W, H, i) for i, (W, H, K) in enumerate(rasters)]
    segs = smoe.Segments([dict(width=W, height=H, num_kernels=K) for W, H, K in rasters])
    assert segs.T // segs.n < 16
    want = [oracle.bin(m, 1, 0, W, H) for m, (W, H, _) in zip(models, rasters)]
    assert max(int(o["counts"].max()) for o in want) > 100
    b = smoe.bin_batched(dev(np.concatenate(models)), 1, 0, segs, capacity=sum(o["P"] for o in want))
    assert not b.read_status()[0]
    at = 0
    for o, sg in zip(want, segs.host):
        at = check(b, len(o["ranges"]), o, sg.tile_offset, sg.kernel_offset, at)
