"""The backward's walk over each kernel's pixels: four list entries a wave, the box of the
entry's ellipse in the block in steps of 1, 2, 4 or 8 rows, entries ordered by their step
counts in chunks of 64.  Gradients against the oracle where that can go wrong: lists of 1, 3, 4,
5, 63, 64, 65 and 130 entries; boxes of one or two columns, of every width and of the whole
block; thin slanted ellipses; kernels that reach no pixel of a listed block; scales 1 and 3 and
window origins; and the same gradient from the fit step, bit for bit.  The bar is the
repository's for gradients (1e-3 of the group's largest; the sums' own rounding is about 1e-6
of it)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.test_gpu_parity import dev, groups, host, say

pytestmark = pytest.mark.gpu
G_TOL = 1e-3

#        name,    K,  C, order, scale, ox, oy, mode
CASES = [("mixed", 1, 3, 1, 1, 0, 0, "smoe"), ("mixed", 3, 3, 1, 1, 0, 0, "smoe"),
         ("mixed", 4, 1, 0, 1, 0, 0, "smoe"), ("mixed", 5, 1, 1, 1, 0, 0, "rbf"),
         ("whole", 63, 3, 1, 1, 0, 0, "smoe"), ("whole", 64, 3, 0, 1, 0, 0, "smoe"),
         ("whole", 65, 3, 1, 1, 0, 0, "smoe"), ("whole", 130, 1, 0, 1, 0, 0, "smoe"),
         ("tiny", 200, 3, 1, 1, 0, 0, "smoe"), ("thin", 120, 3, 1, 1, 0, 0, "smoe"),
         ("thin", 120, 3, 1, 3, 7, 5, "smoe"), ("mixed", 150, 3, 1, 3, 0, 0, "rbf"),
         ("tiny", 90, 1, 0, 2, 3, 0, "smoe")]


def model(kind, K, C, order, W, H, seed):
    m = wl.random_model(K, C, order, W, H, seed, margin=4.0).astype(np.float64)
    rng = np.random.default_rng(seed + 1)
    if kind == "whole":      # every ellipse reaches every block
        m[:, 2:5] = [40.0, 3.0, 45.0]
    elif kind == "tiny":     # a pixel or two, some between the pixel centres
        m[:, 2] = rng.uniform(0.05, 0.6, K)
        m[:, 4] = rng.uniform(0.05, 0.6, K)
        m[:, 3] = rng.uniform(-0.2, 0.2, K)
    elif kind == "thin":     # long slanted needles: a square box full of blocks they miss
        m[:, 2] = rng.uniform(0.3, 9.0, K)
        m[:, 4] = rng.uniform(0.08, 0.5, K)
        m[:, 3] = rng.uniform(-9.0, 9.0, K)
    elif K > 8:              # every size of box
        m[:, 2:5] *= np.exp(rng.uniform(-2.0, 1.0, (K, 1)))
    return m.astype(np.float32)


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}{c[1]}C{c[2]}o{c[3]}s{c[4]}{c[7]}" for c in CASES])
def test_gradient_against_oracle(smoe, case, record_error):
    import torch
    kind, K, C, order, s, ox, oy, mode = case
    say("backward boxes", case)
    W, H = 40, 37
    m_np = model(kind, K, C, order, W, H, 900 + K)
    if mode == "rbf":
        m_np[:, 5] -= 2.0
    OW, OH = s * W - ox, s * H - oy
    rng = np.random.default_rng(K)
    up = rng.normal(size=(OH, OW, C)).astype(np.float32)
    grid = smoe.make_grid(OW, OH, s, ox, oy, mode=mode)
    m = dev(m_np)
    img, D, _, b = smoe.render(m, C, order, grid)
    g = host(smoe.render_backward(m, C, order, grid, b, img, D, grad_image=dev(up)))
    _, g_o = oracle.loss_grad(m_np, C, order, OW, OH, grad_y=up, s=s, ox=ox, oy=oy,
                              rbf=mode == "rbf")
    for name, cols in groups(C, order).items():
        # a kernel alone is its own gate: y = m, so the gates' exact gradient is zero and their
        # rounding is measured by the whole gradient instead
        alone = K == 1 and mode == "smoe"
        peak = max(np.max(np.abs(g_o if alone else g_o[:, cols])), 1e-12)
        e = float(np.max(np.abs(g[:, cols] - g_o[:, cols])) / peak)
        record_error(f"grad {name}", e, G_TOL)
        assert e <= G_TOL, (name, e)
    if s == 1:
        raw = m_np.astype(np.float64)
        raw[:, 2], raw[:, 4] = np.log(raw[:, 2]), np.log(raw[:, 4])
        t = dev(rng.uniform(0, 1, (OH, OW, C)))
        st = smoe.FitState(t, dev(raw), order, smoe.AdamConfig(total_steps=9), max_steps=1, mode=mode)
        rows = st.model.clone()
        img, D, _, b = smoe.render(rows, C, order, grid)
        want = smoe.render_backward(rows, C, order, grid, b, img, D, target=t)
        st.step()
        if int(b.read_status()[1][2]) <= 128:     # (longer lists: the render sums quarters)
            assert torch.equal(st.grads, want)
