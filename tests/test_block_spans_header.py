"""The library's own helpers that say which output blocks a native block is (output_axis,
native_first, native_of, first_block and the binary32 sample coordinate), compiled for the host
from its headers: at every native-block boundary of every scale over the whole accepted range of
o + u, and as rasters use them against a search over the sample coordinates."""
import ctypes as ct
import subprocess

import numpy as np
import pytest

from paper_2510_05814_amd import build

SOURCE = r"""
#include "device_common.h"
using namespace smoe;
extern "C" {
// boundaries at which the last point before or the first point of a native block is not in it
long long boundaries(int scale, int reach, long long* seen) {
  const float inv_s = 1.0f / (float)scale;
  long long bad = 0;
  *seen = 0;
  for (long long b = -(long long)reach / (16 * scale); 16ll * scale * b <= reach; ++b, ++*seen) {
    const int p = (int)(16 * scale * b);
    for (int o = -1; o <= 1; ++o)  // (any split of the coordinate into origin and pixel)
      if (native_block(sample_coord(p - 1 - o, o, inv_s)) != (float)(b - 1) ||
          native_block(sample_coord(p - o, o, inv_s)) != (float)b)
        ++bad;
    if (native_of(first_block(p), scale) != b || native_of(first_block(p - 1), scale) != b - 1) ++bad;
  }
  return bad;
}
int axis(float b0, float b1, int n, int o, int scale, int* out) {
  return output_axis(b0, b1, n, o, scale, 1.0f / (float)scale, out[0], out[1], out[2], out[3]);
}
// per block of an axis: the block that is counted for it
void counted(int n, int o, int scale, int* out) {
  const int b0 = first_block(o);
  for (int t = 0; t < blocks_across(n, o); ++t)
    out[t] = native_first(native_of(b0 + t, scale), scale, b0);
}
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("spans")
    (d / "spans.hip").write_text(SOURCE)
    flags = [f for f in build.FLAGS if not f.startswith("--offload-arch")]
    subprocess.run([build.HIPCC, "--offload-host-only", "--offload-arch=gfx950", *flags, "-shared",
                    str(d / "spans.hip"), "-o", str(d / "spans.so")], check=True,
                   capture_output=True, text=True)
    L = ct.CDLL(str(d / "spans.so"))
    L.boundaries.restype = ct.c_longlong
    L.axis.argtypes = [ct.c_float, ct.c_float, ct.c_int, ct.c_int, ct.c_int, ct.POINTER(ct.c_int)]
    return L


def test_every_boundary(lib):
    reach = (1 << 22) + 65536
    total = 0
    for scale in range(1, 65):
        seen = ct.c_longlong()
        assert lib.boundaries(scale, reach, ct.byref(seen)) == 0, scale
        assert seen.value >= 2 * reach // (16 * scale)
        total += seen.value
    assert total > 2 * 10 ** 6


def test_axes_against_search(lib):
    F = np.float32
    rng = np.random.default_rng(1)
    for t in range(400):
        s = int(rng.integers(1, 65))
        o = int(rng.integers(-(1 << 22), 1 << 22)) if t % 2 else int(rng.integers(-700, 700))
        n = 65536 if t % 40 == 0 else int(np.exp(rng.uniform(0, np.log(65536))))
        u = o + np.arange(n)
        native = np.floor((u.astype(F) + F(0.5)) * (F(1) / F(s)) * F(0.0625)).astype(np.int64)
        block = u // 16 - o // 16
        T = int(block[-1]) + 1
        first = (ct.c_int * T)()
        lib.counted(n, o, s, first)
        starts = np.searchsorted(block, np.arange(T))
        assert np.array_equal(native[starts], native[np.append(starts[1:], n) - 1])  # one native block
        assert np.array_equal(np.array(first), block[np.searchsorted(native, native[starts])])
        for k in range(6):
            b0 = int(rng.integers(native[0] - 2, native[-1] + 2))
            b1 = b0 + int(rng.integers(0, 4)) if k else 1 << 30
            b0 = b0 if k else -(1 << 30)
            at = np.flatnonzero((native >= b0) & (native <= b1))
            out = (ct.c_int * 4)()
            assert bool(lib.axis(b0, b1, n, o, s, out)) == (len(at) > 0)
            if len(at):
                assert list(out) == [block[at[0]], block[at[-1]], native[at[0]], native[at[-1]]]
    out = (ct.c_int * 4)()
    nan, inf = float("nan"), float("inf")
    assert not lib.axis(nan, 1.0, 50, 0, 2, out) and not lib.axis(0.0, nan, 50, 0, 2, out)
    assert lib.axis(-inf, inf, 50, 0, 2, out) and list(out) == [0, 3, 0, 1]
