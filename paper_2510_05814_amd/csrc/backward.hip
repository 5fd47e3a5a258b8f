// Backward (adjoint) of the rasterized SMoE render on gfx950: the standalone call.
//
// Nothing per (pixel, kernel) is stored by the forward: for every pixel the backward
// recomputes each participating kernel's gate term pi K from the record and divides by the
// saved denominator D, then forms the adjoints of all 6 + 3C raw parameters (formulas in
// tile_math.h).  Pixels outside the ellipse or the kernel's blocks contribute nothing
// (Sec. IV-B).
//
// Work split: one wave (four on small rasters) per 16x16 block, four kernels of its list at a time, 16 lanes each; a
// reduction inside the 16 lanes (DPP) leaves one per-(block, kernel) partial row.  A second pass sums each kernel's partial rows over its
// blocks in row-major block order.  Every order is fixed: gradients are bitwise
// reproducible and no atomics are used.
#include "tile_math.h"

namespace smoe {
namespace {

struct BackwardArgs {
  Segs S;
  int C;
  const float* __restrict__ records;
  const int2* __restrict__ ranges;
  const uint32_t* __restrict__ vals;
  const float* __restrict__ image;
  const float* __restrict__ denom;
  const float* __restrict__ grad_image;  // upstream dL/dy, or null
  const float* __restrict__ target;      // MSE target, or null
  float* __restrict__ pair_grads;
};

template <int C, int ORDER, bool RBF, int WAVES>
__global__ __launch_bounds__(kWave * WAVES) void k_backward(BackwardArgs a) {
  constexpr int ROWS = kStrips / WAVES;
  __shared__ PixelSeed<C> seeds[kTilePixels];
  __shared__ __align__(16) BackwardScratch sc;
  const int tile = xcd_block(blockIdx.x, a.S.T);
  const SegGrid sg = seg_of_tile(a.S, tile);
  const PixelCoords<ROWS> px = lane_pixels<WAVES>(sg, tile - sg.tile_offset);
  const int lane = threadIdx.x & 63;
  // MSE of this raster: dL/dy = 2 (y - t) / (W H C)
  const float inv_n2 = 2.0f / ((float)sg.W * (float)sg.H * (float)C);
  const BlockPixels bp = block_pixels<WAVES>(sg, tile - sg.tile_offset);
  const PixelValue<C>* img = reinterpret_cast<const PixelValue<C>*>(a.image) + bp.base;
  const PixelValue<C>* ref =  // the target, or the upstream gradient
      reinterpret_cast<const PixelValue<C>*>(a.target ? a.target : a.grad_image) + bp.base;
  const float* den = a.denom + bp.base;
  float D[ROWS];
  PixelValue<C> y[ROWS], t[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    D[i] = 0.0f;
    if (in_raster(px.u, px.v0 + 4 * i, sg)) {
      const int p = bp.off + i * bp.step;
      D[i] = den[p];
      y[i] = img[p];
      t[i] = ref[p];
    }
  }
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    PixelSeed<C> sd = hole_seed<C>();
    if (D[i] > 0.0f) {
      const float invD = RBF ? 1.0f : __builtin_amdgcn_rcpf(D[i]);
      float gy = 0.0f;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const float g = a.target ? (y[i].v[c] - t[i].v[c]) * inv_n2 : t[i].v[c];
        if (!RBF) gy = __builtin_fmaf(g, y[i].v[c], gy);
        sd.g[c] = g * invD;
      }
      sd.gy = live_gy(gy * invD);
    }
    seeds[((lane >> 4) + 4 * (i + ROWS * wave_index<WAVES>())) * kTile + (lane & 15)] = sd;
  }
  const float2 o = block_base(sg, tile - sg.tile_offset);
  backward_accumulate<C, ORDER, false, WAVES>(block_box(sg, tile - sg.tile_offset), o.x, o.y, sg.inv_s,
                                       a.S.r, a.S.r2, a.records, a.vals, 0, false, a.ranges[tile],
                                       seeds, sc, false, nullptr, a.pair_grads);
}

struct GatherArgs {
  Segs S;
  const float* __restrict__ records;
  const int4* __restrict__ tile_rects;
  const int2* __restrict__ ranges;
  const uint32_t* __restrict__ vals;
  const float* __restrict__ pair_grads;
  const int32_t* __restrict__ status;
  float* __restrict__ grads;
};

// 16 lanes per kernel (one 16-lane row of the wave); lane i ends with parameter i.
template <int C, int ORDER>
__global__ __launch_bounds__(256) void k_gather(GatherArgs a) {
  constexpr int NP = num_params(C, ORDER);
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = gid >> 4, i = gid & 15;
  constexpr int RS = record_stride(C, ORDER);
  const bool live = j < a.S.K;
  const float rec = live && i < RS ? a.records[(size_t)j * RS + i] : 0.0f;
  // every lane takes part in the gather's row reduction and the finishing shuffles
  const float s = gather_param<NP>(j, live && a.status[1] == 0, seg_of_kernel(a.S, live ? j : 0),
                                   a.tile_rects, a.ranges, a.vals, a.pair_grads);
  const float g = finish_gradient<C, ORDER, kRecExpert>(s, live, rec);
  if (live && i < NP) a.grads[(size_t)j * NP + i] = g;
}

}  // namespace

hipError_t launch_backward(int C, int order, const Segs& S, const smoe_bins& b,
                           const float* image, const float* denom, const float* grad_image,
                           const float* target, hipStream_t s) {
  BackwardArgs a{S,
                 C,
                 b.records,
                 reinterpret_cast<const int2*>(b.ranges),
                 b.vals,
                 image,
                 denom,
                 grad_image,
                 target,
                 b.pair_grads};
  with_shape(C, order, S, [&](auto sh) {
    using T = decltype(sh);
    if (S.T <= kSplitBackward)
      k_backward<T::C, T::ORDER, T::RBF, 4><<<S.T, 4 * kWave, 0, s>>>(a);
    else
      k_backward<T::C, T::ORDER, T::RBF, 1><<<S.T, kWave, 0, s>>>(a);
  });
  return hipGetLastError();
}

hipError_t launch_gather(int C, int order, const Segs& S, const smoe_bins& b, float* grads,
                         hipStream_t s) {
  if (S.K == 0) return hipSuccess;
  GatherArgs a{S,
               b.records,
               reinterpret_cast<const int4*>(b.tile_rects),
               reinterpret_cast<const int2*>(b.ranges),
               b.vals,
               b.pair_grads,
               b.status,
               grads};
  const int blocks = (int)(((long long)S.K * 16 + 255) / 256);
  if (C == 1 && order == 0) k_gather<1, 0><<<blocks, 256, 0, s>>>(a);
  else if (C == 1 && order == 1) k_gather<1, 1><<<blocks, 256, 0, s>>>(a);
  else if (C == 3 && order == 0) k_gather<3, 0><<<blocks, 256, 0, s>>>(a);
  else k_gather<3, 1><<<blocks, 256, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace smoe
