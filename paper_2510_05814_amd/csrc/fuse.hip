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
// Each output pixel is summed over the m^2 windows that cover it in (ky, kx) order, in
// binary32, and divided by m^2 (correctly rounded): a gather with one fixed order and no
// atomics, so the fused image is bitwise reproducible.  Every window pixel is read once (m^2 W H
// C floats), W H C floats are written: with many windows a pixel the kernel runs at the rate of
// HBM, with few its launch and the latency of a few loads are what it costs.
#include <type_traits>

#include "device_common.h"

namespace smoe {
namespace {

struct FuseAxis {
  int n, d, w, m;

  __device__ int start(int k) const {
    const int e = (k + 1) * d - w;
    return e > 0 ? e : 0;
  }
  __device__ int len(int k) const { return min(n, (k + 1) * d) - start(k); }
  // sum over i = 1 .. k of min(n, i d) - max(0, i d - w): at most m n < 2^27, taken modulo 2^32
  __device__ int prefix(int k) const {
    const int q = n / d;
    uint32_t s = k <= q ? d * tri(k) : d * tri(q) + (uint32_t)(k - q) * n;
    if (k > m) s -= d * (tri(k) - tri(m)) - (uint32_t)w * (k - m);
    return (int)s;
  }
  __device__ static uint32_t tri(uint32_t k) {
    return k & 1 ? k * ((k + 1) / 2) : (k / 2) * (k + 1);
  }
};

template <int C>
struct Pixel {
  float v[C];
};

// A wave per 64 pixels of an output row.  Straight from a thread per pixel, a load would touch
// another window with every d lanes, a few pixels of each cache line, and fetch each line from
// L2 again for the next window.  So the wave first copies the parts of the windows' rows
// that lie over its pixels to LDS, 2^span lanes a window, whole lines at a time; then each lane
// adds its windows in order from there.  R loads a lane are in flight, and those of
// the next row of windows are issued before this one is added; all of them are unconditional (a
// lane without a pixel copies one that nothing reads: a branch around each takes 55.9 us where
// this takes 41).  Rows of more windows than the wave can hold go in batches.  An odd stride
// between windows spreads the adds over the banks.  512^2, 64 windows a pixel, a thread per
// pixel against this: RGB (204 MB) 59.8 -> 41.0 us, 5.0 TB/s; grey 36.3 -> 19.2; 301 x 203
// RGB 15.2 -> 13.4; 16 windows 12.4 and 12.4, 4 windows 9.5 and 9.2.
constexpr int kFuseWaves = 4;

template <int C, int R>
__global__ __launch_bounds__(64 * kFuseWaves) void k_fuse_windows(const float* __restrict__ win,
                                                                  FuseAxis ax, FuseAxis ay,
                                                                  float hyp, int span,
                                                                  float* __restrict__ out) {
  constexpr int AHEAD = R > 5 ? 8 : 4;
  // a batch: R 2^(6 - span) windows of (C 2^span) | 1 floats
  __shared__ float s_stage[kFuseWaves][R * 64 * (C + 1)];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int x0 = blockIdx.x * 64, x1 = min(ax.n, x0 + 64), x = x0 + lane;
  const int y = blockIdx.y * kFuseWaves + wave;
  if (y >= ay.n) return;  // (no workgroup barriers below)
  float* stage = s_stage[wave];
  const int stride = (C << span) | 1, batch = R << (6 - span);
  const int kx = x / ax.d, ky0 = y / ay.d;
  const int k0 = x0 / ax.d, k1 = (x1 - 1) / ax.d + ax.m - 1;  // the windows over [x0, x1)
  const long long row_pixels = (long long)ax.m * ax.n;
  const int p0 = ax.prefix(k0);

  // what the lane loads of batch kb: rounds of window kb + (r << (6 - span)) + (lane >> span)
  int before[R], len[R], at[R], held = -1;
  auto slots = [&](int kb) {
    if (kb == held) return;
    held = kb;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int k = kb + (r << (6 - span)) + (lane >> span), kc = min(k, k1);
      const int s = ax.start(kc), px = max(s, x0) + (lane & ((1 << span) - 1));
      before[r] = ax.prefix(kc) - p0;
      len[r] = ax.len(kc);
      at[r] = px < min(s + len[r], x1) ? px - s : 0;  // (else a copy that nothing reads)
    }
  };
  Pixel<C> v[R];
  auto load = [&](int ky, int kb) {
    slots(kb);
    const int hy = ay.len(ky), dy = y - ay.start(ky);
    // the first window's pixels of this row of windows, then 32-bit offsets from there
    const Pixel<C>* row =
        reinterpret_cast<const Pixel<C>*>(win) + ay.prefix(ky) * row_pixels + (long long)hy * p0;
#pragma unroll
    for (int r = 0; r < R; ++r)
      v[r] = row[hy * before[r] + dy * len[r] + at[r]];
  };
  float acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0f;
  load(ky0, k0);
  for (int ky = ky0, kb = k0; ky < ky0 + ay.m;) {
    wave_sync();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float* dst = stage + ((r << (6 - span)) + (lane >> span)) * stride +
                   (lane & ((1 << span) - 1)) * C;
#pragma unroll
      for (int c = 0; c < C; ++c) dst[c] = v[r].v[c];
    }
    wave_sync();
    const int done = kb;
    kb += batch;
    if (kb > k1) {
      kb = k0;
      ++ky;
    }
    if (ky < ky0 + ay.m) load(ky, kb);
    const int end = x < x1 ? min(done + batch, kx + ax.m) : 0;
    for (int i0 = max(done, kx); i0 < end; i0 += AHEAD) {
      float u[AHEAD][C];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        const int k = min(i0 + i, end - 1);
        const float* src = stage + (k - done) * stride + (x - max(ax.start(k), x0)) * C;
#pragma unroll
        for (int c = 0; c < C; ++c) u[i][c] = src[c];
      }
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        if (i0 + i < end) {
#pragma unroll
          for (int c = 0; c < C; ++c) acc[c] += u[i][c];
        }
      }
    }
  }
  if (x >= x1) return;
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
  const dim3 grid((width + 63) / 64, (height + kFuseWaves - 1) / kFuseWaves);
  int span = 0;  // lanes a window: 2^span
  while (span < 6 && (1 << span) < window) ++span;
  const float hyp = (float)((long long)m * m);
  // rounds of copies that the windows over 64 pixels take (ten for all: 16.8 us where five take
  // 12.4 with 16 windows a pixel, 11.4 where three take 9.2 with 4)
  const int windows_over = 63 / d + (64 % d ? 1 : 0) + m;
  const int rounds = (windows_over + (1 << (6 - span)) - 1) >> (6 - span);
  auto launch = [&](auto r) {
    constexpr int R = decltype(r)::value;
    if (C == 1)
      k_fuse_windows<1, R><<<grid, 64 * kFuseWaves, 0, s>>>(windows, ax, ay, hyp, span, image);
    else
      k_fuse_windows<3, R><<<grid, 64 * kFuseWaves, 0, s>>>(windows, ax, ay, hyp, span, image);
  };
  if (rounds <= 3) launch(std::integral_constant<int, 3>{});
  else if (rounds <= 5) launch(std::integral_constant<int, 5>{});
  else launch(std::integral_constant<int, 10>{});
  return hipGetLastError();
}

}  // namespace smoe
