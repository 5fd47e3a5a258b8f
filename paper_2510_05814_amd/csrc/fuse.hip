// Multi-model fusion of block-overlapping window models (Sec. V-C, Eq. (10)-(11)) on gfx950.
//
// Along an axis of n pixels, window k of size w shifted by the displacement d covers
// [max(0, (k+1)d - w), min(n, (k+1)d)): the first window starts w - d pixels before the
// image, and every pixel x lies in exactly m = w/d windows per axis, k = floor(x/d) ...
// floor(x/d) + m - 1.  The window renders arrive concatenated in window order (rows of
// windows top to bottom, each row left to right), each window's clipped pixels row-major with
// C channels interleaved.  Since every row of windows holds m n_x pixels per image row, the
// start of window (ky, kx) is prefix_y(ky) m n_x + len_y(ky) prefix_x(kx), with prefix(k) the
// pixels of windows 0 .. k-1 of an axis, in closed form.
//
// One thread per output pixel sums the m^2 windows that cover it in (ky, kx) order, in
// binary32, and divides by m^2 (correctly rounded): a gather with one fixed order and no
// atomics, so the fused image is bitwise reproducible.  The kernel is HBM bound: every window
// pixel is read once (m^2 W H C floats), W H C floats are written.
#include "smoe_internal.h"

namespace smoe {
namespace {

struct FuseAxis {
  int n, d, w, m;

  __device__ int start(int k) const {
    const int e = (k + 1) * d - w;
    return e > 0 ? e : 0;
  }
  __device__ int len(int k) const { return min(n, (k + 1) * d) - start(k); }
  // sum over i = 1 .. k of min(n, i d) - max(0, i d - w)
  __device__ long long prefix(int k) const {
    const long long q = n / d, kk = k;
    long long s = kk <= q ? d * (kk * (kk + 1) / 2) : d * (q * (q + 1) / 2) + (kk - q) * n;
    if (kk > m) s -= d * (kk * (kk + 1) / 2 - (long long)m * (m + 1) / 2) - (long long)w * (kk - m);
    return s;
  }
};

template <int C>
struct Pixel {
  float v[C];
};

// A thread per output pixel, 64 x 4 of them a workgroup.  Along a row of windows the position of
// the pixel moves from window to window by the earlier one's size and the change of its row's
// start: a few 32-bit operations a window.  The loads of AHEAD windows are issued before the
// first is added (RGB: one 12-byte load a window); the sum keeps its order.  512^2 RGB, 64
// windows a pixel (204 MB): 76.6 -> 59.9 us against 64-bit positions worked out and three 4-byte
// loads waited for in every window.
template <int C>
__global__ __launch_bounds__(256) void k_fuse_windows(const float* __restrict__ win, FuseAxis ax,
                                                      FuseAxis ay, float hyp,
                                                      float* __restrict__ out) {
  constexpr int AHEAD = 8;
  const int x = blockIdx.x * 64 + (threadIdx.x & 63);
  const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (x >= ax.n || y >= ay.n) return;
  const long long row_pixels = (long long)ax.m * ax.n;
  const int kx0 = x / ax.d, ky0 = y / ay.d;
  const long long px0 = ax.prefix(kx0);
  float acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0f;
  for (int ky = ky0; ky < ky0 + ay.m; ++ky) {
    const int hy = ay.len(ky), dy = y - ay.start(ky);
    // the first window's pixels of this row of windows, then offsets from there
    const Pixel<C>* row = reinterpret_cast<const Pixel<C>*>(win) + ay.prefix(ky) * row_pixels + hy * px0;
    int before = 0;  // pixels of the windows passed
    for (int i0 = 0; i0 < ax.m; i0 += AHEAD) {
      Pixel<C> v[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        if (i0 + i < ax.m) {
          const int s = ax.start(kx0 + i0 + i), wx = ax.len(kx0 + i0 + i);
          v[i] = row[before + dy * wx + (x - s)];
          before += hy * wx;
        }
      }
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        if (i0 + i < ax.m) {
#pragma unroll
          for (int c = 0; c < C; ++c) acc[c] += v[i].v[c];
        }
      }
    }
  }
  Pixel<C> o;
#pragma unroll
  for (int c = 0; c < C; ++c) o.v[c] = acc[c] / hyp;
  reinterpret_cast<Pixel<C>*>(out)[(long long)y * ax.n + x] = o;
}

}  // namespace

hipError_t launch_fuse_windows(const float* windows, int C, int width, int height, int window,
                               int d, float* image, hipStream_t s) {
  const int m = window / d;
  const FuseAxis ax{width, d, window, m}, ay{height, d, window, m};
  const dim3 grid((width + 63) / 64, (height + 3) / 4);
  const float hyp = (float)((long long)m * m);
  if (C == 1) k_fuse_windows<1><<<grid, 256, 0, s>>>(windows, ax, ay, hyp, image);
  else k_fuse_windows<3><<<grid, 256, 0, s>>>(windows, ax, ay, hyp, image);
  return hipGetLastError();
}

}  // namespace smoe
