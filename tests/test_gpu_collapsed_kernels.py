"""Kernels collapsed to lines thinner than binary32 can divide by: no pixel lies inside such an
ellipse, so its gradient is zero -- not 0 * inf -- and the other kernels' is what it is without
it.  Fit step and standalone backward, one chunk of entries and several, against the oracle; the
bar is the repository's for gradients (1e-3 of the group's largest)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, groups, host, say

pytestmark = pytest.mark.gpu
G_TOL = 1e-3

#            l11, l21, l22: 1/l11 near the largest number; 1/l22; the ratio l21/l22
COLLAPSED = [(2e-38, 4.0, 3.0), (6e-39, -3.0, 5.0), (4.0, 3.0, 2e-38), (5.0, 1e6, 2e-33)]


@pytest.mark.parametrize("K", [12, 50, 120])
@pytest.mark.parametrize("W,H", [(70, 45), (640, 656)])         # four waves a block, one
@pytest.mark.parametrize("trunc", ["gradient", "render"])
def test_gradient_is_zero(trunc, W, H, K, record_error):
    import paper_2510_05814_amd as smoe
    say("collapsed", trunc, W, H, K)
    m_np = wl.random_model(K, 3, 1, 70, 45, K, sig_lo=4.0, sig_hi=9.0, margin=0.0)
    at = np.arange(len(COLLAPSED)) * (K // 4)
    m_np[at, 2:5] = COLLAPSED
    m_np[at, 0:2] = [[20.3, 20.2], [33.1, 18.7], [50.2, 30.4], [25.7, 28.9]]
    t_np = np.random.default_rng(K).uniform(0, 1, (H, W, 3)).astype(np.float32)
    raw = m_np.astype(np.float64)
    raw[:, 2], raw[:, 4] = np.log(raw[:, 2]), np.log(raw[:, 4])
    T = smoe.tiles(W, H)
    st = smoe.FitState(dev(t_np), dev(raw), 1, smoe.AdamConfig(total_steps=9), max_steps=1,
                       trunc=trunc, capacity=T * (K + 16))
    rows = st.model.clone()
    assert (rows[at, 2:5:2] > 0).all()
    grid = smoe.make_grid(W, H, trunc=trunc)
    img, D, _, b = smoe.render(rows, 3, 1, grid)
    g = host(smoe.render_backward(rows, 3, 1, grid, b, img, D, target=dev(t_np)))
    _, g_o = oracle.loss_grad(host(rows), 3, 1, W, H, target=t_np, trunc=trunc)
    assert not g_o[at].any()
    st.step()
    for what, got in (("backward", g), ("fit", host(st.grads))):
        assert not got[at].any(), what
        for name, cols in groups(3, 1).items():
            peak = max(np.max(np.abs(g_o[:, cols])), 1e-12)
            e = float(np.max(np.abs(got[:, cols] - g_o[:, cols])) / peak)
            record_error(f"{what} {name}", e, G_TOL)
            assert e <= G_TOL, (what, name, e)
    assert np.isfinite(host(st.raw)).all()
