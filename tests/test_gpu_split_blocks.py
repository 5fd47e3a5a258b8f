"""Four waves per block on small rasters, one on larger ones: the two give the same bits.  A
raster of 2116 blocks (one wave each) against windows of it and against single images of a
batch (four waves each): renders, denominators, losses, gradients and Adam states equal."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


@pytest.mark.parametrize("C,order,mode,trunc", [(3, 1, "smoe", "gradient"), (1, 0, "rbf", "gradient"),
                                                (3, 0, "smoe", "render"), (1, 1, "smoe", "render")])
def test_windows_and_batches_are_the_same_bits(smoe, C, order, mode, trunc):
    import torch
    say("split blocks", C, order, mode, trunc)
    side = 736
    m = dev(wl.random_model(3000, C, order, side, side, 80 + C + order, sig_lo=1.0, sig_hi=14.0))
    full, D, _, _ = smoe.render(m, C, order, smoe.make_grid(side, side, mode=mode, trunc=trunc))
    assert smoe.tiles(side, side) > 1536
    for ox, oy, w, h in [(0, 0, 333, 301), (16, 32, 16, 16), (401, 390, 335, 346)]:
        img, d, _, _ = smoe.render(m, C, order, smoe.make_grid(w, h, 1, ox, oy, mode=mode, trunc=trunc))
        assert torch.equal(img, full[oy:oy + h, ox:ox + w]) and torch.equal(d, D[oy:oy + h, ox:ox + w])
    # two images together (2116 + 36 blocks) and alone
    rng = np.random.default_rng(5)
    tg, raws = [], []
    for n, K in ((side, 3000), (96, 140)):
        r = wl.random_model(K, C, order, n, n, n, sig_lo=1.0, sig_hi=9.0).astype(np.float64)
        r[:, 2], r[:, 4] = np.log(r[:, 2]), np.log(r[:, 4])
        raws.append(dev(r))
        tg.append(dev(rng.uniform(0, 1, (n, n, C))))
    kw = dict(mode=mode, trunc=trunc, max_steps=2)
    both = smoe.FitState(tg, raws, order, smoe.AdamConfig(total_steps=9), **kw)
    alone = smoe.FitState(tg[1], raws[1], order, smoe.AdamConfig(total_steps=9), **kw)
    for _ in range(2):
        both.step()
        alone.step()
    torch.cuda.synchronize()
    assert torch.equal(both.raw_rows()[1], alone.raw) and torch.equal(both.images()[1], alone.image)
    assert torch.equal(both.grads[3000:], alone.grads) and torch.equal(both.v[3000:], alone.v)
    assert torch.equal(both.segment_losses()[1:], alone.segment_losses())
    # the render's loss, its backward and the fit step's on either side
    for n, t, raw in ((side, tg[0], raws[0]), (96, tg[1], raws[1])):
        st = smoe.FitState(t, raw, order, smoe.AdamConfig(total_steps=9), **kw)
        rows, grid = st.model.clone(), smoe.make_grid(n, n, mode=mode, trunc=trunc)
        img, d, _, b = smoe.render(rows, C, order, grid, target=t)
        g = smoe.render_backward(rows, C, order, grid, b, img, d, target=t)
        st.step()
        assert torch.equal(st.image, img) and torch.equal(st.grads, g)
