"""The render's two ways of forming a term's exponent (entries of a block that may pass the
representable range, and the others): blocks whose corners lie between -60 and -300 of a listed
kernel's exponent, so that entries fall on both sides of the test and pixels on both sides of
the cut at -125.  Images within 1e-5, D within its bar, and the same pixels covered, against
the oracle; lists of one and of several entries, one and three channels, scales 1 and 2."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests._tol import d_rel_error
from tests.test_gpu_parity import D_RTOL, Y_TOL, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smoe():
    import paper_2510_05814_amd as smoe
    return smoe


@pytest.mark.parametrize("K,C,order,s", [(1, 3, 1, 1), (6, 1, 0, 1), (40, 3, 0, 1), (24, 3, 1, 2),
                                         (90, 1, 1, 1)])
def test_far_entries_against_oracle(smoe, K, C, order, s, record_error):
    say("far entries", K, C, order, s)
    W = H = 16 * int(np.ceil(2.2 * np.sqrt(K))) + 16     # about one kernel per five blocks
    rng = np.random.default_rng(50 + K)
    m_np = wl.random_model(K, C, order, W, H, 60 + K, margin=0.0).astype(np.float64)
    # standard deviations of 0.75 to 2 px: 16 pixels away the exponent is -46 to -330
    m_np[:, 2] = rng.uniform(0.75, 2.0, K)
    m_np[:, 4] = rng.uniform(0.75, 2.0, K)
    m_np[:, 3] = rng.uniform(-0.5, 0.5, K)
    m_np[:, 5] = rng.uniform(-3.0, 3.0, K)
    m_np = m_np.astype(np.float32)
    m = dev(m_np)
    img, D, _, _ = smoe.render(m, C, order, smoe.make_grid(s * W, s * H, s))
    y_o, D_o = oracle.render(m_np, C, order, s * W, s * H, s)
    assert (D_o == 0).any() and (D_o > 0).any() and np.any((D_o > 0) & (np.log2(D_o + (D_o == 0)) < -110))
    assert np.array_equal(host(D) > 0, D_o > 0)
    ey = float(np.max(np.abs(host(img) - y_o)))
    eD = d_rel_error(host(D), D_o)
    record_error("image abs", ey, Y_TOL)
    record_error("D rel", eD, D_RTOL)
    assert ey <= Y_TOL and eD <= D_RTOL
