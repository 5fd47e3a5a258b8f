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
// C floats), W H C floats are written.  Two kernels, the same bits: straight from the windows, a
// thread per pixel (k_fuse_pixels), or by way of LDS where a load of 64 neighbouring pixels would
// touch too many windows (k_fuse_windows; by_lds has the rule and both sides' times).
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
// between windows spreads the adds over the banks.  It runs at the rate of HBM (512^2 RGB, 64
// windows a pixel, 204 MB: 38.3 to 41 us).
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

// A thread per output pixel.  Along a row of windows the position of the pixel moves from window to
// window by the earlier one's size and the change of its row's start: a few 32-bit operations a
// window.  The loads of AHEAD windows are issued before the first is added.  A load instruction
// touches another window with every d lanes: with few windows a pixel the launch and the latency of
// a few loads are what it costs, with many windows and a small d the lines it fetches again.
template <int C, int AHEAD>
__global__ __launch_bounds__(64 * kFuseWaves) void k_fuse_pixels(const float* __restrict__ win,
                                                                 FuseAxis ax, FuseAxis ay,
                                                                 float hyp,
                                                                 float* __restrict__ out) {
  const int x = blockIdx.x * 64 + (threadIdx.x & 63);
  const int y = blockIdx.y * kFuseWaves + (threadIdx.x >> 6);
  if (x >= ax.n || y >= ay.n) return;
  const long long row_pixels = (long long)ax.m * ax.n;
  const int kx0 = x / ax.d, ky0 = y / ay.d;
  const int px0 = ax.prefix(kx0);
  float acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0f;
  for (int ky = ky0; ky < ky0 + ay.m; ++ky) {
    const int hy = ay.len(ky), dy = y - ay.start(ky);
    // the first window's pixels of this row of windows, then 32-bit offsets from there
    const Pixel<C>* row =
        reinterpret_cast<const Pixel<C>*>(win) + ay.prefix(ky) * row_pixels + (long long)hy * px0;
    int before = 0;  // pixels of the windows passed (at most 1024^3)
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

// Whether windows of w pixels, shifted by d, go by way of LDS.  Measured, a thread per pixel / LDS:
// 512^2 RGB at (w, d) = (16, 2) 42 / 38 us, (8, 1) 74 / 49, (16, 1) 414 / 195, (32, 1) 1753 / 960,
// (8, 2) 13.1 / 12.2 and grey (16, 2) 33 / 19, 1024^2 RGB (32, 2) 1000 / 861 -- but (64, 2) 907 /
// 1150, (16, 4) 11.7 / 12.5, (24, 3) 38 / 75, (16, 8) 4.9 / 7.0, (16, 16) 4.3 / 6.0, (2, 1) 4.9 / 6.8,
// grey (64, 8) 18 / 71 and 2048^2 RGB (16, 8) 39 / 52, (16, 16) 22 / 42.  RGB window renders that
// exceed the last-level cache go by LDS at larger d too: 2048^2 (16, 4) 180 / 158, (15, 5) 106 / 95,
// 1200^2 (16, 4) 54 / 51 (1024^2: 35.7 / 36.9; grey 2048^2: 63 / 84; RGB (20, 5) 181 / 189).
constexpr long long kLastLevelCache = 256ll << 20;
inline bool by_lds(int C, int width, int height, int w, int d) {
  const int m = w / d;
  if (d <= 2) return m >= 4 && (d == 1 || w <= 32);
  return C == 3 && m >= 3 && w <= 16 &&
         (long long)m * m * width * height * C * (long long)sizeof(float) > kLastLevelCache;
}

}  // namespace

hipError_t launch_fuse_windows(const float* windows, int C, int width, int height, int window,
                               int d, float* image, hipStream_t s) {
  const int m = window / d;
  const FuseAxis ax{width, d, window, m}, ay{height, d, window, m};
  const dim3 grid((width + 63) / 64, (height + kFuseWaves - 1) / kFuseWaves);
  const float hyp = (float)((long long)m * m);
  if (by_lds(C, width, height, window, d)) {
    int span = 0;  // lanes a window: 2^span
    while (span < 6 && (1 << span) < window) ++span;
    // rounds of copies that the windows over 64 pixels take: five or ten in flight
    const int windows_over = 63 / d + (64 % d ? 1 : 0) + m;
    const int rounds = (windows_over + (1 << (6 - span)) - 1) >> (6 - span);
    auto launch = [&](auto r) {
      constexpr int R = decltype(r)::value;
      if (C == 1)
        k_fuse_windows<1, R><<<grid, 64 * kFuseWaves, 0, s>>>(windows, ax, ay, hyp, span, image);
      else
        k_fuse_windows<3, R><<<grid, 64 * kFuseWaves, 0, s>>>(windows, ax, ay, hyp, span, image);
    };
    if (rounds <= 5) launch(std::integral_constant<int, 5>{});
    else launch(std::integral_constant<int, 10>{});
    return hipGetLastError();
  }
  auto launch = [&](auto ahead) {
    constexpr int AHEAD = decltype(ahead)::value;
    if (C == 1) k_fuse_pixels<1, AHEAD><<<grid, 64 * kFuseWaves, 0, s>>>(windows, ax, ay, hyp, image);
    else k_fuse_pixels<3, AHEAD><<<grid, 64 * kFuseWaves, 0, s>>>(windows, ax, ay, hyp, image);
  };
  if (m == 1) launch(std::integral_constant<int, 1>{});
  else if (m == 2) launch(std::integral_constant<int, 2>{});
  else if (m <= 4) launch(std::integral_constant<int, 4>{});
  else launch(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

}  // namespace smoe
