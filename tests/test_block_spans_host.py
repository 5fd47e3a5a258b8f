"""The closed form of an axis' output blocks (native block b is the 16 s output pixels from 16 s b
on) against a search over the binary32 sample coordinates, over the accepted range of origins,
sizes and scales."""
import numpy as np

F = np.float32


def test_native_block_pixels_closed_form():
    rng = np.random.default_rng(0)
    for t in range(600):
        s = int(rng.integers(1, 65))
        o = int(rng.integers(-(1 << 22), 1 << 22)) if t % 2 else int(rng.integers(-500, 500))
        n = 65536 if t % 50 == 0 else int(np.exp(rng.uniform(0, np.log(65536))))
        inv_s = F(1) / F(s)
        block = np.floor(((o + np.arange(n)).astype(F) + F(0.5)) * inv_s * F(0.0625)).astype(np.int64)
        for _ in range(4):
            b0 = int(rng.integers(block[0], block[-1] + 1))
            b1 = int(rng.integers(b0, block[-1] + 1))
            at = np.flatnonzero((block >= b0) & (block <= b1))
            assert at[0] == max(0, 16 * s * b0 - o), (s, o, n, b0)
            assert at[-1] == min(n - 1, 16 * s * (b1 + 1) - 1 - o), (s, o, n, b1)
