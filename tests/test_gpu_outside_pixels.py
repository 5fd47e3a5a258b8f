"""Gradients of blocks with pixels that get none: those that hang over the edge of an odd-sized
raster, and pixels whose denominator the caller hands over as zero.  The kernels here stay finite
at every other pixel and leave binary32 at those -- a centre outside the raster with a mixing weight
near the largest (the term itself, or its product with dy, passes the range) -- so whatever such a
pixel still added would be 0 * inf.  Standalone backward and fit step, one wave a block and four,
both expert orders, against the oracle; the bar is the repository's for gradients (1e-3 of the
group's largest)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, groups, host, say

pytestmark = pytest.mark.gpu
G_TOL = 1e-3


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


def model(kind, order, W, H, extra=0):
    """Some ordinary kernels and, last, one centred outside the right edge."""
    m = wl.random_model(40 + extra, 3, order, W, H, 77, sig_lo=2.0, sig_hi=5.0, margin=0.0)
    k = m[-1]
    k[6:] = 0.0
    k[6:9] = [0.3, 0.6, 0.4]
    if kind == "term":       # 2^128 within 0.7 sigma of the centre, at most 2^102 in the raster
        k[:6] = [W + 8.0, H / 2.0, 1.4, 0.0, 4.0, 89.0]
    else:                    # exp(87.13) = 7e37: dy K passes the range near the centre's column only
        k[:6] = [W + 8.0, H / 2.0, 1.4, 0.0, 20.0, 87.13]
    return m


#                                        blocks: 6 (four waves), 1599 (fit: one), 6241 (both: one)
@pytest.mark.parametrize("W,H,extra", [(33, 17, 0), (641, 609, 4000), (1249, 1249, 4000)])
@pytest.mark.parametrize("kind,order", [("term", 0), ("term", 1), ("product", 1)])
def test_pixels_outside_the_raster(smoe, kind, order, W, H, extra, record_error):
    say("outside pixels", kind, order, W, H)
    m_np = model(kind, order, W, H, extra)
    rng = np.random.default_rng(W)
    t_np = rng.uniform(0, 1, (H, W, 3)).astype(np.float32)
    raw = m_np.astype(np.float64)
    raw[:, 2], raw[:, 4] = np.log(raw[:, 2]), np.log(raw[:, 4])
    st = smoe.FitState(dev(t_np), dev(raw), order, smoe.AdamConfig(total_steps=9), max_steps=1)
    rows = st.model.clone()
    grid = smoe.make_grid(W, H)
    img, D, _, b = smoe.render(rows, 3, order, grid)
    g = host(smoe.render_backward(rows, 3, order, grid, b, img, D, target=dev(t_np)))
    assert np.isfinite(host(img)).all() and np.isfinite(host(D)).all()
    _, g_o = oracle.loss_grad(host(rows), 3, order, W, H, target=t_np)
    assert np.isfinite(g_o).all()
    st.step()
    for what, got in (("backward", g), ("fit", host(st.grads))):
        assert np.isfinite(got).all(), what
        for name, cols in groups(3, order).items():
            peak = max(np.max(np.abs(g_o[:, cols])), 1e-12)
            e = float(np.max(np.abs(got[:, cols] - g_o[:, cols])) / peak)
            record_error(f"{what} {name}", e, G_TOL)
            assert e <= G_TOL, (what, name, e)
    for t in (st.raw, st.m, st.v, st.model):
        assert np.isfinite(host(t)).all()
    assert int(st.bins.read_status()[1][3]) == 0


@pytest.mark.parametrize("mode", ["smoe", "rbf"])
def test_pixels_the_caller_leaves_out(smoe, mode):
    """denom = 0: whatever stands in the image and the gradient there takes no part."""
    import torch
    say("left out", mode)
    W, H = 40, 37
    m = dev(wl.random_model(90, 3, 1, W, H, 5, sig_lo=1.0, sig_hi=6.0))
    grid = smoe.make_grid(W, H, mode=mode)
    img, D, _, b = smoe.render(m, 3, 1, grid)
    up = dev(np.random.default_rng(3).normal(size=(H, W, 3)))
    out = torch.zeros((H, W), dtype=torch.bool, device="cuda")
    out[3:20, 5:18] = out[36, :] = out[:, 39] = True
    D = torch.where(out, torch.zeros_like(D), D)
    zeroed = torch.where(out[..., None], torch.zeros_like(up), up)
    bad = torch.where(out[..., None], torch.full_like(up, float("nan")), up)
    want = smoe.render_backward(m, 3, 1, grid, b, img, D, grad_image=zeroed)
    got = smoe.render_backward(m, 3, 1, grid, b, img, D, grad_image=bad)
    assert torch.isfinite(want).all() and torch.equal(got, want)
