// Per-block math of the rasterized SMoE on gfx950, shared by the standalone render and
// backward calls and the fused fit-step kernel.  Internal header.
//
// Lane layout of the forward: a block is four 16x4 strips, strip i the rows (l >> 4) + 4i of
// lane l, which owns column l & 15.  One wave takes all four strips -- the column's terms
// (dx, z1, l21 z1, z1^2) are then computed once per kernel for four pixels -- or, on rasters of
// too few blocks to fill the chip that way, four waves take a strip each (WAVES).  Either way a
// pixel's sums are formed by one lane over the whole list in the same operations, so the
// results are the same bits.
#pragma once

#include <type_traits>

#include "device_common.h"

namespace smoe {

constexpr int kWave = 64;

// Compile-time shape of a launch: channels, expert order, regression mode (RBF: the
// un-normalised sum of Eq. 1 instead of the gated SMoE of Eq. 2-4) and the reading of the
// truncation (which bound the render applies).
template <int C_, int ORDER_, bool RBF_, int TRUNC_>
struct Shape {
  static constexpr int C = C_, ORDER = ORDER_, TRUNC = TRUNC_;
  static constexpr bool RBF = RBF_;
};

// Calls f(Shape<...>{}) for the run-time (C, order, mode, reading); C is 1 or 3, order 0 or 1.
template <int C, int ORDER, class F>
inline void with_mode(const Segs& S, F&& f) {
  const bool rbf = S.mode == SMOE_MODE_RBF;
  if (S.trunc == SMOE_TRUNC_RENDER)
    rbf ? f(Shape<C, ORDER, true, SMOE_TRUNC_RENDER>{}) : f(Shape<C, ORDER, false, SMOE_TRUNC_RENDER>{});
  else
    rbf ? f(Shape<C, ORDER, true, SMOE_TRUNC_GRADIENT>{})
        : f(Shape<C, ORDER, false, SMOE_TRUNC_GRADIENT>{});
}
template <class F>
inline void with_shape(int C, int order, const Segs& S, F&& f) {
  if (C == 1 && order == 0) with_mode<1, 0>(S, f);
  else if (C == 1 && order == 1) with_mode<1, 1>(S, f);
  else if (C == 3 && order == 0) with_mode<3, 0>(S, f);
  else with_mode<3, 1>(S, f);
}
constexpr int kChunk = 64;                     // records staged in LDS per chunk
constexpr int kStrips = kTilePixels / kWave;   // 16x4 strips of a block (4)

// Waves per block: one, or four (a strip each) on rasters whose blocks alone leave SIMDs idle
// (1024 of them).  Four waves pay the column's terms four times over, one per SIMD waits on
// its own latencies.  Measured, one wave against four, at 1024 / 1369 / 1521 / 1600 / 1764 / 2025
// blocks: RGB linear render 12.8 / 12.9 / 13.2 / 13.5 / 14.2 / 14.8 us against 10.5 / 12.8 / 13.1 /
// 13.6 / 14.9 / 16.1, fit step 31.9 / 31.7 / 33.0 / 31.8 / 34.2 / 34.4 against 27.3 / 28.5 / 29.2 /
// 32.0 / 33.0 / 35.1; grey constant render 10.8 / - / 11.0 / - / 11.6 / 11.9 against 7.6 / - / 8.8 / -
// / 9.4 / 10.3, fit step 28.1 / - / 28.6 / - / 29.8 / 30.1 against 22.4 / - / 23.9 / - / 25.8 / 29.2.  The
// backward alone has no such terms (its groups of entries are dealt out whole): 15.9 us against
// 12.8 at 1024 blocks, 23.6 against 23.4 at 3600, 30.2 against 28.8 at 5184, 37.1 against 37.9 at
// 7744.
// Batches of small rasters (few_blocks) mostly give four waves nothing to share: one (a fit of 1392
// windows of a block each 22.6 us against 23.5).
constexpr int kSplitForward = 1536, kSplitBackward = 6144;
inline bool split_blocks(const Segs& S) { return S.T <= kSplitForward && !few_blocks(S); }

// The wave's index in its workgroup, wave-uniform.
template <int WAVES>
__device__ __forceinline__ int wave_index() {
  return WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// ROWS: the lane's pixels, one per strip its wave takes.
template <int ROWS>
struct PixelCoords {
  int u;            // output column of the lane (within its raster; < 0 or >= W: outside)
  int v0;           // output row of the lane's first pixel (rows v0 + 4i)
  float x;          // sampling coordinates
  float y[ROWS];
};

// A pixel's C channel values, moved as one load or store of 4 C bytes.  RGB: one 12-byte
// access instead of three strided by 12, each of which touches every line again; with the
// fit's four target loads in flight together, its 2048^2 step 114.6 -> 111.3 us, a fit of
// 16641 one-block windows that stores its render 98.1 -> 89.8 us, bin + render of the 2048^2
// model 83.7 -> 81.4 us.
template <int C>
struct PixelValue {
  float v[C];
};

// Where a block's pixels lie in the concatenated images: its first pixel (before the buffer's
// start where the block hangs over the raster) and the lane's first one relative to it, rows
// 4 raster rows apart -- 32-bit offsets from a wave-uniform base.
struct BlockPixels {
  long long base;
  int off, step;
};

// Whether output pixel (u, v) lies in the raster (the first and last blocks of a window may
// hang over its edges).
__device__ __forceinline__ bool in_raster(int u, int v, const SegGrid& g) {
  return (unsigned)u < (unsigned)g.W && (unsigned)v < (unsigned)g.H;
}

// `tile` is the block index inside the segment's raster.  The raster's blocks are aligned
// to multiples of 16 in the output coordinate o + u (SegGrid), so the block's first column
// is u = 16 (bx0 + tx) - ox.  A native block is 16 s output pixels and begins on such a
// multiple (binary32 sample coordinates included, over the whole accepted range of origins,
// sizes and scales), so all of a block's points lie in one native block and every kernel of
// its list is a member at every one of them: no per-point membership test.
template <int WAVES>
__device__ __forceinline__ PixelCoords<kStrips / WAVES> lane_pixels(const SegGrid& g, int tile) {
  constexpr int ROWS = kStrips / WAVES;
  PixelCoords<ROWS> p;
  const int lane = threadIdx.x & 63;
  const int tx = tile % g.ntx, ty = tile / g.ntx;
  p.u = kTile * (g.bx0 + tx) - g.ox + (lane & 15);
  p.v0 = kTile * (g.by0 + ty) - g.oy + (lane >> 4) + 4 * ROWS * wave_index<WAVES>();
  p.x = sample_coord(p.u, g.ox, g.inv_s);
#pragma unroll
  for (int i = 0; i < ROWS; ++i) p.y[i] = sample_coord(p.v0 + 4 * i, g.oy, g.inv_s);
  return p;
}

template <int WAVES>
__device__ __forceinline__ BlockPixels block_pixels(const SegGrid& g, int tile) {
  const int lane = threadIdx.x & 63;
  const int u = kTile * (g.bx0 + tile % g.ntx) - g.ox, v = kTile * (g.by0 + tile / g.ntx) - g.oy;
  const int row = (lane >> 4) + 4 * (kStrips / WAVES) * wave_index<WAVES>();
  return BlockPixels{g.pixel_offset + (long long)v * g.W + u, row * g.W + (lane & 15), 4 * g.W};
}

// A wave-uniform value moved to a scalar register (it then holds no vector register over the
// loops between its uses).
__device__ __forceinline__ float in_sgpr(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// Coordinates of a block's first and last column and row (whole blocks, also where they hang
// over the raster's edges).
struct BlockBox {
  float x0, x1, y0, y1;
  float scale;  // rows per unit of y
};
__device__ __forceinline__ BlockBox block_box(const SegGrid& g, int tile) {
  const int u = kTile * (g.bx0 + tile % g.ntx) - g.ox, v = kTile * (g.by0 + tile / g.ntx) - g.oy;
  return BlockBox{in_sgpr(sample_coord(u, g.ox, g.inv_s)),
                  in_sgpr(sample_coord(u + kTile - 1, g.ox, g.inv_s)),
                  in_sgpr(sample_coord(v, g.oy, g.inv_s)),
                  in_sgpr(sample_coord(v + kTile - 1, g.oy, g.inv_s)), in_sgpr((float)g.scale)};
}
// o + 0.5 + (column, row) of the block's first pixel (exact): its pixel (c, r) samples
// ((.x + c) * inv_s, (.y + r) * inv_s).
__device__ __forceinline__ float2 block_base(const SegGrid& g, int tile) {
  return make_float2((float)(kTile * (g.bx0 + tile % g.ntx)) + 0.5f,
                     (float)(kTile * (g.by0 + tile / g.ntx)) + 0.5f);
}

// The thread's index, opaque to the compiler: what the once-per-chunk code derives from it is
// then computed there instead of being held in registers across the loops over entries.
__device__ __forceinline__ int local_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Stages the records of list entries [base, base + n) (n <= kChunk) into LDS, with all threads
// of the workgroup.  An entry holds the kernel id shifted left by `shift` (the fit step's
// packed bucket entries; 0 elsewhere).
template <int RS, int WAVES>
__device__ __forceinline__ void stage_records(float4* __restrict__ srec,
                                              const float* __restrict__ records,
                                              const uint32_t* __restrict__ vals, int base, int n,
                                              int shift) {
  constexpr int Q = RS / 4;
  __syncthreads();
  for (int i = local_thread(); i < n * Q; i += kWave * WAVES) {
    const int k = i / Q, c = i - k * Q;
    srec[i] = reinterpret_cast<const float4*>(records + (size_t)(vals[base + k] >> shift) * RS)[c];
  }
  __syncthreads();
}

// The same by way of ent, LDS room for the chunk's entries.
template <int RS, int WAVES>
__device__ __forceinline__ void stage_records_lds(float4* __restrict__ srec,
                                                  const float* __restrict__ records,
                                                  const uint32_t* __restrict__ vals, int base,
                                                  int n, int shift, uint32_t* __restrict__ ent) {
  constexpr int Q = RS / 4;
  __syncthreads();
  const int t = local_thread();
  if (t < n) ent[t] = vals[base + t];
  __syncthreads();
  for (int i = local_thread(); i < n * Q; i += kWave * WAVES) {
    const int k = i / Q, c = i - k * Q;
    srec[i] = reinterpret_cast<const float4*>(records + (size_t)(ent[k] >> shift) * RS)[c];
  }
  __syncthreads();
}

// A render record of RS floats into registers.
template <int RS>
__device__ __forceinline__ void load_record(float (&r)[RS], const float4* __restrict__ f4) {
#pragma unroll
  for (int k = 0; k < RS / 4; ++k) {
    const float4 f = f4[k];
    r[4 * k] = f.x;
    r[4 * k + 1] = f.y;
    r[4 * k + 2] = f.z;
    r[4 * k + 3] = f.w;
  }
}

// Entries of a staged chunk for which some pixel of the block may lie beyond the render's
// representable range (exponent below -125): bit k for entry k < n.  A lane per entry: the
// exponent is least where q is largest, and q, a convex function of the point, is largest at
// a corner of the block; the bound -110 instead of -125 covers every rounding.  Blocks near
// their kernels have no such entry.
template <int RS>
__device__ __forceinline__ uint64_t far_entries(const BlockBox& bb, const float4* srec, int n) {
  const int lane = local_thread() & 63;
  bool far = false;
  if (lane < n) {
    const float4 f = srec[lane * (RS / 4)], g = srec[lane * (RS / 4) + 1];
    const float za = (bb.x0 - f.x) * f.z, zb = (bb.x1 - f.x) * f.z;
    const float ta = f.w * za, tb = f.w * zb, d0 = bb.y0 - f.y, d1 = bb.y1 - f.y;
    const float a0 = (d0 - ta) * g.x, a1 = (d1 - ta) * g.x, b0 = (d0 - tb) * g.x, b1 = (d1 - tb) * g.x;
    const float qa = za * za + fmaxf(a0 * a0, a1 * a1), qb = zb * zb + fmaxf(b0 * b0, b1 * b1);
    const float ea = __builtin_fmaf(qa, -0.5f * kLog2e, g.y), eb = __builtin_fmaf(qb, -0.5f * kLog2e, g.y);
    far = !(ea >= -110.0f) || !(eb >= -110.0f);
  }
  return __ballot(far);
}

// One list entry of the forward: its terms pi K (e) and expert values m_c at the lane's pixels,
// e = 0 where the render's rule drops the term; D = sum pi K, N_c = sum pi K m_c.  TRUNC == SMOE_TRUNC_RENDER: the
// ellipse q <= r^2.  TRUNC == SMOE_TRUNC_GRADIENT (the block lists decide the render): every
// term binary32 holds, i.e. whose exponent a = rho log2(e) - q log2(e)/2 is >= -125.  r: the
// entry's render record; cut_scale, cut_offset: the render's bound in the compare-free form of
// Segs; far: whether some pixel of the block may lie beyond that bound.
//
// The loop over entries is bound by VALU issue: a binary32 add, multiply or fma on vector
// registers takes 2 cycles of a SIMD, a compare, select, min or max, or an operand in a scalar
// register 4, exp2 8.  So an entry that is not far -- almost all of them -- takes its exponent
// straight as a = alpha - v^2 with v = (dy - t) sqrt(log2(e)/2) / l22 and alpha = rho log2(e)
// - z1^2 log2(e)/2, the column's part: four operations a pixel instead of six and a minimum,
// and no compare.  Otherwise the decisions are taken on the ABI's own binary32 sequence, and
// the bound goes through the exponent: with the ellipse, max(q, u) with u = fma(q,
// cut_scale, cut_offset) is q inside the bound and gives a term beyond it an exponent of about
// -2^36; with the representable range, min(a, fma(a, 2^60, 125 * 2^60)) is a for a >= -125 and
// below -2^43 otherwise: exp2 of an excluded term is exactly zero.
// Measured: binning and render of a 2048^2 model with 65536 kernels 88.5 -> 83.7 us, its fit
// step 116.1 -> 114.6 us, a 512^2 render with lists of several hundred 332 -> 320 us.
template <int C, int ORDER, int TRUNC, int ROWS>
__device__ __forceinline__ void entry_terms(const PixelCoords<ROWS>& px, float r2, float cut_scale,
                                            float cut_offset,
                                            const float (&r)[record_stride(C, ORDER)], bool far,
                                            float (&e)[ROWS], float (&m)[ROWS][C]) {
  const float dx = px.x - r[0];
  const float z1 = dx * r[2];
  const float tt = r[3] * z1;
  const float zz1 = z1 * z1;
  // a_c + wx_c dx: the expert's value along the lane's column
  float mx[C];
#pragma unroll
  for (int c = 0; c < C; ++c)
    mx[c] = ORDER == 1 ? __builtin_fmaf(r[kRecExpert + C + c], dx, r[kRecExpert + c])
                       : r[kRecExpert + c];
  float dy[ROWS], a[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) dy[i] = px.y[i] - r[1];
  // pi K = exp(rho - q/2) = exp2(rho log2 e - q log2 e / 2)
  if (TRUNC == SMOE_TRUNC_GRADIENT && !far) {
    constexpr float kRoot = 0.84932180028801904272f;  // sqrt(log2(e) / 2)
    const float kk = r[4] * kRoot;
    const float alpha = __builtin_fmaf(zz1, -0.5f * kLog2e, r[5]);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const float v = (dy[i] - tt) * kk;
      a[i] = __builtin_fmaf(-v, v, alpha);
    }
  } else {
    float q[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const float w = dy[i] - tt;
      const float z2 = w * r[4];
      q[i] = zz1 + z2 * z2;
    }
    if (TRUNC == SMOE_TRUNC_RENDER) {
      // (the bound is the identity, bit for bit, where every pixel lies inside: four pixels a
      // lane ask first, one applies it)
      bool out = ROWS == 1;
      if (ROWS > 1) {
        float qmax = q[0];
#pragma unroll
        for (int i = 1; i < ROWS; ++i) qmax = __builtin_fmaxf(qmax, q[i]);
        out = __any(!(qmax <= r2));
      }
      if (out) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
          q[i] = __builtin_fmaxf(q[i], __builtin_fmaf(q[i], cut_scale, cut_offset));
      }
#pragma unroll
      for (int i = 0; i < ROWS; ++i) a[i] = __builtin_fmaf(q[i], -0.5f * kLog2e, r[5]);
    } else {
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        a[i] = __builtin_fmaf(q[i], -0.5f * kLog2e, r[5]);
        a[i] = __builtin_fminf(a[i], __builtin_fmaf(a[i], cut_scale, cut_offset));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    e[i] = __builtin_amdgcn_exp2f(a[i]);
#pragma unroll
    for (int c = 0; c < C; ++c)
      m[i][c] = ORDER == 1 ? __builtin_fmaf(r[kRecExpert + 2 * C + c], dy[i], mx[c]) : mx[c];
  }
}

// The terms of one entry added to the pixels' sums.
template <int C, int ROWS>
__device__ __forceinline__ void add_terms(const float (&e)[ROWS], const float (&m)[ROWS][C],
                                          float (&D)[ROWS], float (&N)[ROWS][C]) {
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    D[i] += e[i];
#pragma unroll
    for (int c = 0; c < C; ++c) N[i][c] = __builtin_fmaf(e[i], m[i][c], N[i][c]);
  }
}

// The entries of a staged chunk, in order.
template <int C, int ORDER, int TRUNC, int ROWS>
__device__ __forceinline__ void forward_chunk(const PixelCoords<ROWS>& px, const BlockBox& bb, float r2,
                                              float cut_scale, float cut_offset,
                                              const float4* srec, int n, float (&D)[ROWS],
                                              float (&N)[ROWS][C]) {
  constexpr int RS = record_stride(C, ORDER);
  constexpr int Q = RS / 4;
  const uint64_t far = TRUNC == SMOE_TRUNC_GRADIENT ? far_entries<RS>(bb, srec, n) : 0;
  auto one = [&](int k) {
    float r[RS], e[ROWS], m[ROWS][C];
    load_record<RS>(r, &srec[k * Q]);
    entry_terms<C, ORDER, TRUNC, ROWS>(px, r2, cut_scale, cut_offset, r, (far >> k & 1) != 0, e, m);
    add_terms<C, ROWS>(e, m, D, N);
  };
  int k = 0;
  if (ROWS == 1) {
    // one strip to a wave: an entry is one chain of dependent operations and few waves share
    // the SIMD, so AHEAD entries are formed side by side and then added in order (with the
    // records' loading during the ranking, four steps of a 64^2 grey fit 88.3 -> 77.9 us)
    constexpr int AHEAD = 4;
    for (; k + AHEAD <= n; k += AHEAD) {
      if ((far >> k & ((1u << AHEAD) - 1)) != 0) {
        for (int i = 0; i < AHEAD; ++i) one(k + i);
        continue;
      }
      float r[AHEAD][RS], e[AHEAD][ROWS], m[AHEAD][ROWS][C];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) load_record<RS>(r[i], &srec[(k + i) * Q]);
#pragma unroll
      for (int i = 0; i < AHEAD; ++i)
        entry_terms<C, ORDER, TRUNC, ROWS>(px, r2, cut_scale, cut_offset, r[i], false, e[i], m[i]);
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) add_terms<C, ROWS>(e[i], m[i], D, N);
    }
  }
  for (; k < n; ++k) one(k);
}

// A copy of x that the compiler must keep in a vector register: loop-invariant operands of
// the forward's per-row arithmetic are read from VGPRs rather than SGPRs (see entry_terms).
__device__ __forceinline__ float in_vgpr(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <int C, int ROWS>
__device__ __forceinline__ void zero_sums(float (&D)[ROWS], float (&N)[ROWS][C]) {
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    D[i] = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) N[i][c] = 0.0f;
  }
}

// Forward accumulation over a block's list [rg.x, rg.y) in list order (forward_chunk per
// chunk, records staged through LDS in chunks).
// shift: list entries hold the kernel id << shift.  ent: null, or LDS room for one chunk of
// entries for the staging to go by.  staged: the list is one chunk and its records stand in
// srec already.
template <int C, int ORDER, int TRUNC, int WAVES>
__device__ __forceinline__ void forward_accumulate(const PixelCoords<kStrips / WAVES>& px, const BlockBox& bb,
                                                   float r2, float cut_scale, float cut_offset,
                                                   const float* __restrict__ records,
                                                   const uint32_t* __restrict__ vals, int shift,
                                                   int2 rg, float4* srec, float (&D)[kStrips / WAVES],
                                                   float (&N)[kStrips / WAVES][C],
                                                   uint32_t* ent = nullptr,
                                                   bool staged = false) {
  constexpr int RS = record_stride(C, ORDER);
  zero_sums<C>(D, N);
  if (TRUNC == SMOE_TRUNC_RENDER) {
    cut_scale = in_vgpr(cut_scale);
    cut_offset = in_vgpr(cut_offset);
  }
  for (int base = rg.x; base < rg.y; base += kChunk) {
    const int n = __builtin_amdgcn_readfirstlane(min(kChunk, rg.y - base));
    if (staged) {
      // (nothing to load)
    } else if (ent) stage_records_lds<RS, WAVES>(srec, records, vals, base, n, shift, ent);
    else stage_records<RS, WAVES>(srec, records, vals, base, n, shift);
    forward_chunk<C, ORDER, TRUNC, kStrips / WAVES>(px, bb, r2, cut_scale, cut_offset, srec, n, D, N);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// Transposed reduction inside each 16-lane row: on return lane l holds the sum over the
// row's 16 lanes of v[l & 15].  Stages pair lane l with l ^ 8 (row_ror:8), with 7 - l in its
// group of 8 (row_half_mirror), then l ^ 2 and l ^ 1 (quad_perm); at each stage a lane keeps
// the half of its values selected by that bit of its index and adds the partner's copy.
// Every lane of the row must be active.
__device__ __forceinline__ float row_reduce16_transposed(float (&v)[16]) {
  const int lane = threadIdx.x & 63;
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0, b1 = (lane & 2) != 0,
             b0 = (lane & 1) != 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float keep = b3 ? v[i + 8] : v[i], send = b3 ? v[i] : v[i + 8];
    v[i] = keep + dpp<0x128>(send);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = b2 ? v[i + 4] : v[i], send = b2 ? v[i] : v[i + 4];
    v[i] = keep + dpp<0x141>(send);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b1 ? v[i + 2] : v[i], send = b1 ? v[i] : v[i + 2];
    v[i] = keep + dpp<0x4E>(send);
  }
  const float keep = b0 ? v[1] : v[0], send = b0 ? v[0] : v[1];
  return keep + dpp<0xB1>(send);
}

// Adds partial row p (NP values of a row of partial_stride(NP) floats) to v.
template <int NP>
__device__ __forceinline__ void add_partial_row(float (&v)[16], const float* __restrict__ pair_grads,
                                                int p) {
  constexpr int PS = partial_stride(NP);
  const float4* row = reinterpret_cast<const float4*>(pair_grads + (size_t)p * PS);
#pragma unroll
  for (int q4 = 0; q4 < PS / 4; ++q4) {
    const float4 x = row[q4];
    if (4 * q4 + 0 < NP) v[4 * q4 + 0] += x.x;
    if (4 * q4 + 1 < NP) v[4 * q4 + 1] += x.y;
    if (4 * q4 + 2 < NP) v[4 * q4 + 2] += x.z;
    if (4 * q4 + 3 < NP) v[4 * q4 + 3] += x.w;
  }
}

// The position of kernel j in block t's sorted list (a binary search; entries hold the
// kernel id << shift), or -1 if the list does not hold j.
__device__ __forceinline__ int list_position(int j, int t, const int2* __restrict__ ranges,
                                             const uint32_t* __restrict__ vals, int shift) {
  const int2 rg = ranges[t];
  if (rg.y <= rg.x) return -1;
  return find_in_list(vals, rg.x, rg.y, (uint32_t)j, shift);
}

// Gradient of kernel row j: the sum of its per-block partial rows over its block rectangle.
// A group of 16 lanes (one 16-lane row of the wave) serves one kernel: lane b adds the partial
// rows of blocks b, b + 16, ... of the rectangle (row-major); the row reduction then leaves
// parameter i's gradient in lane i.  The summation order is fixed, so the result is
// reproducible.  The standalone backward's partial row of a (block, kernel) pair is at the
// pair's list position, found by a search.  All 16 lanes must call it (live = false: the
// kernel contributes nothing).
template <int NP>
__device__ __forceinline__ float gather_param(int j, bool live, const SegGrid& sg,
                                              const int4* __restrict__ rects,
                                              const int2* __restrict__ ranges,
                                              const uint32_t* __restrict__ vals,
                                              const float* __restrict__ pair_grads) {
  static_assert(NP <= 16, "16 lanes per kernel");
  float v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) v[q] = 0.0f;
  if (live) {
    const int4 rc = rects[j];
    const int n = rect_count(rc);
    const int w = rc.z - rc.x + 1;
    for (int b = threadIdx.x & 15; b < n; b += 16) {
      const int dy = b / w;
      const int p = list_position(j, sg.tile_offset + (rc.y + dy) * sg.ntx + rc.x + (b - dy * w),
                                  ranges, vals, 0);
      if (p >= 0) add_partial_row<NP>(v, pair_grads, p);
    }
  }
  return row_reduce16_transposed(v);
}

// The fit step's gather, in the same order, with the kernel's rectangle rc already loaded by
// the caller.  The partial row of the kernel's block b is at row kSlots j + b for b < kSlots
// (contiguous per kernel); beyond, at row kSlots K + the bucket slot that the entry's low bits
// hold, found by a search of the block's sorted list.
template <int NP>
__device__ __forceinline__ float gather_param_fit(int j, bool live, const Segs& S, int4 rc,
                                                  const int2* __restrict__ ranges,
                                                  const uint32_t* __restrict__ vals,
                                                  const float* __restrict__ pair_grads,
                                                  int shift) {
  static_assert(NP <= 16, "16 lanes per kernel");
  float v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) v[q] = 0.0f;
  if (live) {
    const int n = rect_count(rc);
    const int w = rc.z - rc.x + 1;
    for (int b = threadIdx.x & 15; b < n; b += 16) {
      int p = j * kSlots + b;
      if (b >= kSlots) {
        const SegGrid sg = seg_of_kernel(S, j);
        const int dy = b / w;
        const int t = sg.tile_offset + (rc.y + dy) * sg.ntx + rc.x + (b - dy * w);
        const int pos = list_position(j, t, ranges, vals, shift);
        if (pos < 0) continue;
        const int low = (int)(vals[pos] & ((1u << shift) - 1u));
        p = S.K * kSlots + ranges[t].x + (low - kSlots);
      }
      add_partial_row<NP>(v, pair_grads, p);
    }
  }
  return row_reduce16_transposed(v);
}

// A kernel's gradient from the sums of its partial rows (lane i of the kernel's 16-lane group
// holds the sum of field i; every lane of the group must call it).  Fields 0 and 1 of a
// partial row leave out the expert terms of the centre's gradient, which factor through the
// kernel's slopes and are applied here once per kernel:
//   dL/dmu_x = field 0 - sum_c wx_c dL/da_c,  dL/dmu_y = field 1 - sum_c wy_c dL/da_c.
// slopes: a per-lane value whose lane SLOPES + C + c holds wx_c and lane SLOPES + 2C + c
// holds wy_c (the render record's fields, or the kernel's raw row: the same numbers).
template <int C, int ORDER, int SLOPES>
__device__ __forceinline__ float finish_gradient(float s, bool live, float slopes) {
  if (ORDER == 0) return s;
  const int i = threadIdx.x & 15;
  float ex = 0.0f;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const float da = __shfl(s, 6 + c, 16);
    const float slope = __shfl(slopes, SLOPES + ((i == 0) ? 1 : 2) * C + c, 16);
    ex = __builtin_fmaf(da, slope, ex);
  }
  return live && i < 2 ? s - ex : s;
}

// The sum over each 16-lane row of 16 values, as row_reduce16_transposed (lane l ends with the
// row's sum of v[l & 15]), for values the caller has just computed.  The first two stages add
// with the DPP lane mask doing the selection: for the pair (v[i], v[i + 8]) one add leaves
// v[i] + v[i](l ^ 8) in every lane and a second, written only to lanes 8-15 of the row
// (bank_mask 0xc), replaces it there by v[i + 8] + v[i + 8](l ^ 8) -- two 4-cycle adds per pair
// instead of two selects and an add.  DPP reads of a register need two wait states after
// its write, which nothing inserts inside an asm block: the leading and trailing s_nop and the
// order of the adds (a register is read at least five instructions after its write) give
// them.  Every lane of the wave must be active.
__device__ __forceinline__ float row_reduce16_masked(float (&v)[16]) {
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %12, %12 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %5, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %6, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %6, %14, %14 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %7, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %7, %15, %15 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %3, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 1"
      : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3]), "+&v"(v[4]), "+&v"(v[5]), "+&v"(v[6]),
        "+&v"(v[7])
      : "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]),
        "v"(v[15]));
  const int lane = threadIdx.x & 63;
  const bool b1 = (lane & 2) != 0, b0 = (lane & 1) != 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b1 ? v[i + 2] : v[i], send = b1 ? v[i] : v[i + 2];
    v[i] = keep + dpp<0x4E>(send);
  }
  const float keep = b0 ? v[1] : v[0], send = b0 ? v[0] : v[1];
  return keep + dpp<0xB1>(send);
}

// A block's squared error from the strips' (err: the lane's, of the strips its wave takes): per
// lane ((strip 0 + 1) + (2 + 3)), then a butterfly over the lanes -- one order however many
// waves take the block.  Returns it in every lane of wave 0.  part: kTilePixels floats of LDS
// (unused by one wave); every thread calls it.
template <int WAVES>
__device__ __forceinline__ float block_error(const float (&err)[kStrips / WAVES], float* part) {
  float e[kStrips];
  if (WAVES == 1) {
#pragma unroll
    for (int i = 0; i < kStrips; ++i) e[i] = err[i % (kStrips / WAVES)];
  } else {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < kStrips / WAVES; ++i)
      part[(wave_index<WAVES>() * (kStrips / WAVES) + i) * kWave + lane] = err[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kStrips; ++i) e[i] = part[i * kWave + lane];
  }
  float t = (e[0] + e[1]) + (e[2] + e[3]);
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
  return t;
}

// Adjoint seeds of a block's pixels in LDS, row-major: dL/dy_c / D and sum_c dL/dy_c y_c / D.
// With the seed 1/D -> 1 and
// sum_c g_c y_c -> 0 the same backward is the adjoint of the un-normalised sum of Eq. (1):
// then w = pi K is dy_c/dm_c and G = sum_c g_c m_c is dL/d(pi K).
// A hole is a pixel where no gradient flows (D = 0 or outside the raster).  Zero seeds do not
// always keep it out: a kernel centred outside the raster may pass the range of binary32 there, and
// 0 * inf is not zero.  Its gy is -0, which no other pixel's is (live_gy), for the backward's
// second look.
template <int C>
struct alignas(C == 3 ? 16 : 8) PixelSeed {
  float g[C];
  float gy;
  __device__ bool hole() const { return __float_as_uint(gy) == 0x80000000u; }
};
template <int C>
__device__ __forceinline__ PixelSeed<C> hole_seed() {
  PixelSeed<C> sd;
#pragma unroll
  for (int c = 0; c < C; ++c) sd.g[c] = 0.0f;
  sd.gy = -0.0f;
  return sd;
}
// The gy of a pixel that is no hole: +0 for -0, every other value as it is.
__device__ __forceinline__ float live_gy(float gy) { return gy + 0.0f; }

// The rows [row0, row1] and columns [col0, col1] (of 0..15; empty when row0 > row1) of a block
// that hold every pixel inside the ellipse q <= r^2 of one kernel.  In z1 = (x - mu_x) / l11
// the ellipse's upper edge l21 z1 + l22 sqrt(r^2 - z1^2) is concave, its lower edge convex, so
// over the block's columns each reaches furthest at its extremum clamped to them; the left
// and right edges over the block's rows alike.  r is widened by 1e-3 of itself and by what the
// rounding of dy - l21 z1 can move z2 = (dy - l21 z1) / l22 by, and the edges by a hundredth of
// a pixel and the rounding of the coordinates, far above the error of the binary32 test and
// of this; kernels whose factors leave binary32's comfortable range, and
// whatever compares as not a number, keep the whole block.
struct EllipseBox {
  int row0, row1, col0, col1;
};
__device__ __forceinline__ EllipseBox ellipse_box(const BlockBox& bb, float r, float mux, float muy,
                                                  float i11, float l21, float i22) {
  const float l11 = __builtin_amdgcn_rcpf(i11), l22 = fabsf(__builtin_amdgcn_rcpf(i22));
  const float dx0 = bb.x0 - mux, dx1 = bb.x1 - mux, d0 = bb.y0 - muy, d1 = bb.y1 - muy;
  const float za = fminf(dx0 * i11, dx1 * i11), zb = fmaxf(dx0 * i11, dx1 * i11);
  const float zmax = fminf(fmaxf(fabsf(za), fabsf(zb)), 1.001f * r);
  const float rr =
      1.001f * r + 1e-6f * (fmaxf(fabsf(d0), fabsf(d1)) + fabsf(l21) * zmax) * fabsf(i22);
  const float syy = l21 * l21 + l22 * l22;
  const float is = __builtin_amdgcn_rsqf(syy);
  EllipseBox e{0, 15, 0, 15};
  if (!(syy > 1e-24f && syy < 1e24f && fabsf(l11) > 1e-12f && fabsf(l11) < 1e12f && rr < 1e9f))
    return e;
  // rows: over z1 in [za, zb] cut to [-rr, rr]
  const float zl = fmaxf(za, -rr), zh = fminf(zb, rr);
  const float zs = rr * l21 * is;  // where the upper edge peaks; the lower edge's is -zs
  const float zu = fminf(fmaxf(zs, zl), zh), zd = fminf(fmaxf(-zs, zl), zh);
  const float up = l21 * zu + l22 * __builtin_amdgcn_sqrtf(fmaxf(rr * rr - zu * zu, 0.0f));
  const float dn = l21 * zd - l22 * __builtin_amdgcn_sqrtf(fmaxf(rr * rr - zd * zd, 0.0f));
  const float my = 0.01f + 3e-7f * fmaxf(fabsf(bb.y0), fabsf(bb.y1)) * bb.scale;
  const float t0 = (dn - d0) * bb.scale - my, t1 = (up - d0) * bb.scale + my;
  // columns: over dy in [d0, d1] cut to the ellipse's own extent
  const float ext = rr * syy * is;
  const float dl = fmaxf(d0, -ext), dh = fminf(d1, ext);
  const float ds = rr * l21;  // where the right edge peaks; the left edge's is -ds
  const float du = fminf(fmaxf(ds, dl), dh), dd = fminf(fmaxf(-ds, dl), dh);
  const float e2 = ext * ext, iss = is * is;
  const float zr = (l21 * du + l22 * __builtin_amdgcn_sqrtf(fmaxf(e2 - du * du, 0.0f))) * iss;
  const float zq = (l21 * dd - l22 * __builtin_amdgcn_sqrtf(fmaxf(e2 - dd * dd, 0.0f))) * iss;
  const float xr = fmaxf(zr * l11, zq * l11), xl = fminf(zr * l11, zq * l11);
  const float mx = 0.01f + (3e-7f * fmaxf(fabsf(bb.x0), fabsf(bb.x1)) + 1e-3f * rr * fabsf(l11)) * bb.scale;
  const float c0 = (xl - dx0) * bb.scale - mx, c1 = (xr - dx0) * bb.scale + mx;
  if (t0 > 0.0f) e.row0 = (int)fminf(ceilf(t0), 16.0f);
  if (t1 < 15.0f) e.row1 = (int)fmaxf(floorf(t1), -1.0f);
  if (c0 > 0.0f) e.col0 = (int)fminf(ceilf(c0), 16.0f);
  if (c1 < 15.0f) e.col1 = (int)fmaxf(floorf(c1), -1.0f);
  if (zl > zh || dl > dh || e.col0 > e.col1) e.row0 = 16;
  return e;
}

// Scratch of the backward in LDS, beside the pixel seeds.
struct BackwardScratch {
  uint32_t ent[kChunk];  // the chunk's list entries, then packed boxes
  uint2 out[kChunk];     // (kernel id or staged record, partial row) in processing order
};

// The partial row of a list entry (Backward, below) at position pos of the lists; list0: the
// first position of its list.
__device__ __forceinline__ uint32_t partial_row(uint32_t e, int shift, bool packed, int pos, int K,
                                                int list0) {
  if (!packed) return (uint32_t)pos;
  const uint32_t low = e & ((1u << shift) - 1u);
  return low < (uint32_t)kSlots ? (e >> shift) * (uint32_t)kSlots + low
                                : (uint32_t)K * kSlots + (uint32_t)list0 + (low - kSlots);
}

// One wave lays out the backward of a chunk of n <= 64 entries, a lane per entry (lanes from n
// on pass anything): f, i22 = its record's first fields, at = where its record is, row = its
// partial row.  Leaves in sc, in processing order, the box of pixels its ellipse reaches as
// first row | first column << 4 | log2 rows per step << 8 | pairs of steps << 12, and (at, row).
__device__ __forceinline__ void lay_out_entries(const BlockBox& bb, float radius, int n, float4 f,
                                                float i22, uint32_t at, uint32_t row,
                                                BackwardScratch& sc) {
  const int lane = threadIdx.x & 63;
  int its = 0, packed_box = 0;
  if (lane < n) {
    const EllipseBox b = ellipse_box(bb, radius, f.x, f.y, f.z, f.w, i22);
    if (b.row0 <= b.row1) {
      const int lw = max(1, 32 - __clz(b.col1 - b.col0));  // columns <= 2^lw
      const int lr = 4 - lw;                               // 2^lr rows per step
      its = (b.row1 - b.row0 + (2 << lr)) >> (lr + 1);
      // (the last steps' rows and columns stay inside the block)
      packed_box = min(b.row0, 16 - (its << (lr + 1))) | min(b.col0, 16 - (1 << lw)) << 4 |
                   lr << 8 | its << 12;
    }
  }
  // place by step count (8 .. 0), most first, ties in the lanes' order
  int to = 0, before = 0;
#pragma unroll
  for (int v = 8; v >= 0; --v) {
    const uint64_t same = __ballot(lane < n && its == v);
    const int place = (int)__builtin_amdgcn_mbcnt_hi(
        (uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, (uint32_t)before));
    to = its == v ? place : to;
    before += __popcll(same);
  }
  const uint32_t first = __builtin_amdgcn_readfirstlane(at);
  if (lane >= n) {  // padding, after every entry: its lanes work on the first one's record
    to = lane;
    at = first;
  }
  sc.ent[to] = (uint32_t)packed_box;
  sc.out[to] = make_uint2(at, row);
}

// Backward over a block's list [rg.x, rg.y): for every kernel the adjoints of its 6 + 3C raw
// parameters, summed over the block's 256 pixels (pi K recomputed from the record, w = pi K /
// D), written as the per-(block, kernel) partial row.
//   G = sum_c g_c (m_c - y_c),  H = w G                       (dL/drho)
//   dL/da_c = g_c w,  dL/dwx_c = g_c w dx,  dL/dwy_c = g_c w dy
//   bz2 = -H z2,  bz1 = -H z1 - bz2 l21/l22                  (through q = z1^2 + z2^2)
//   dL/dmu_x = -(bz1/l11 + sum_c g_c w wx_c),  dL/dmu_y = -(bz2/l22 + sum_c g_c w wy_c)
//   dL/ds1 = -bz1 z1,  dL/dl21 = -bz2 z1/l22,  dL/ds2 = -bz2 z2
// Fields 0 and 1 of the partial row leave out the sum_c g_c w wx_c and sum_c g_c w wy_c
// terms: the gather applies them per kernel from dL/da_c (finish_gradient).
//
// What bounds it is VALU issue: a binary32 add, multiply or fma on vector registers takes 2
// cycles of a SIMD here, every other vector instruction (compare, select, DPP, integer) 4,
// exp2 and the permlane swaps 8.  So a wave takes four list entries at a time, 16 lanes
// each, and a lane keeps one column of its entry while it steps down the block's rows: dx,
// z1, what factors through them, the per-lane finish and the reduction are paid once per four
// entries.  (One entry per wave, four rows per lane and a 64-lane reduction paid as much for
// those as for the pairs.)  The 16 lanes cover the box of the entry's ellipse in the
// block (ellipse_box, a lane per entry, 64 entries at once): a box of at most 8, 4 or 2
// columns takes 2, 4 or 8 rows per step.  Entries are taken in the order of their step
// counts (in pairs of steps), most first, so the four of a group need about as many; with
// several waves to a block, they take the groups in turn.
// Measured against one entry per wave: the 2048^2 RGB linear fit step 145 -> 117 us (65536
// kernels, 26-entry lists), the standalone backward of a 509x381 render 20.3 -> 13.7 us.
// The seeds sit in LDS; a lane reads its entry's record from memory, or, where the forward's
// records still stand beside the seeds (staged, lists of one chunk), from there.
//
// Per lane, over its pixels: the sums that do not factor through the column -- A_c =
// sum g_c w, Y_c = sum g_c w dy, V = sum H (dy - t), S2 = sum H z2^2, R = sum H.  dx and z1 are
// the same for the lane's pixels, so sum g_c w dx = dx A_c, sum bz2 = -V / l22 (z2 = (dy - t)
// / l22), sum bz1 = -(z1 R + (l21/l22) sum bz2), sum bz1 z1 = z1 sum bz1.  The seeds are
// divided by D, so w = pi K / D is e = pi K.
// packed (the fit step): list entries hold kernel id << shift | low, and the partial row of
// the entry is row kSlots j + low for low < kSlots (the block's index in the kernel's
// rectangle: kernel-major rows), else row kSlots K + rg.x + low - kSlots (its bucket slot),
// where the fit step's gather reads it; otherwise the entry's list position.
// x0, y0: o + 0.5 + (column, row) of the block's first pixel, whose coordinates are these
// times inv_s; UNIT: inv_s = 1.  laid_out: the list is one chunk and sc holds its layout
// (lay_out_entries); staged: null, or where its records stand in LDS, by the layout's places.
template <int C, int ORDER, bool UNIT, int WAVES>
__device__ __forceinline__ void backward_accumulate(const BlockBox& bb, float x0, float y0,
                                                    float inv_s, float radius, float r2,
                                                    const float* __restrict__ records,
                                                    const uint32_t* __restrict__ vals, int shift,
                                                    bool packed, int2 rg,
                                                    const PixelSeed<C>* seeds, BackwardScratch& sc,
                                                    bool laid_out, const float4* staged,
                                                    float* __restrict__ pair_grads, int K = 0) {
  constexpr int RS = record_stride(C, ORDER);
  constexpr int Q = RS / 4;
  constexpr int NP = num_params(C, ORDER);
  constexpr int PS = partial_stride(NP);
  static_assert(PS <= 16, "16 accumulators per kernel");
  const int lane = threadIdx.x & 63;
  const int l16 = lane & 15, sub = lane >> 4, wave = wave_index<WAVES>();
  for (int base = rg.x; base < rg.y; base += kChunk) {
    const int n = __builtin_amdgcn_readfirstlane(min(kChunk, rg.y - base));
    __syncthreads();
    if (!laid_out) {
      if (wave == 0) {
        const uint32_t e = lane < n ? vals[base + lane] : 0u;
        const float4* r4 = reinterpret_cast<const float4*>(records + (size_t)(e >> shift) * RS);
        float4 f = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float i22 = 0.0f;
        if (lane < n) {
          f = r4[0];
          i22 = r4[1].x;
        }
        lay_out_entries(bb, radius, n, f, i22, e >> shift,
                        partial_row(e, shift, packed, base + lane, K, rg.x), sc);
      }
      __syncthreads();
    }
    for (int g = 4 * wave; g < n; g += 4 * WAVES) {
      const uint32_t bx = sc.ent[g + sub];
      const uint2 out = sc.out[g + sub];
      const int M = __builtin_amdgcn_readfirstlane(bx >> 12);  // the group's first has the most
      float tot = 0.0f;
      // A first look at the group's pixels and, if a sum is no number, a second: 0 * inf may have
      // come from a hole, or from a lane without a pixel and an infinite z1 or reciprocal.  (Flags
      // asked in the first look cost every group: 2048^2 fit step 109.8 -> 111.5 us with them, 108.6
      // -> 109.3 with this.)
      for (bool careful = false; M > 0; careful = true) {
        float r[RS];
        load_record<RS>(r, staged ? staged + out.x * Q
                                  : reinterpret_cast<const float4*>(records + (size_t)out.x * RS));
        const int lr = (int)(bx >> 8 & 7u), mine = (int)(bx >> 12);
        const int col = (int)(bx >> 4 & 15u) + (l16 & ((16 >> lr) - 1));
        const int row0 = (int)(bx & 15u) + (l16 >> (4 - lr));
        const PixelSeed<C>* sp = seeds + row0 * kTile + col;
        float h = y0 + (float)row0;
        const float hstep = (float)(1 << lr);
        const float xc = x0 + (float)col;
        const float dx = (UNIT ? xc : xc * inv_s) - r[0];
        float z1 = dx * r[2];
        const float tt = r[3] * z1;
        const float zz1 = z1 * z1;
        // a_c + wx_c dx: the expert's value along the lane's column
        float mx[C];
#pragma unroll
        for (int c = 0; c < C; ++c)
          mx[c] = ORDER == 1 ? __builtin_fmaf(r[kRecExpert + C + c], dx, r[kRecExpert + c])
                             : r[kRecExpert + c];
        float A[C], Y[C];
#pragma unroll
        for (int c = 0; c < C; ++c) A[c] = Y[c] = 0.0f;
        float V = 0.0f, S2 = 0.0f, R = 0.0f;
        auto walk = [&](auto second_look) {
          for (int m = 0; m < M; ++m) {
            if (m < mine) {
              // both steps' seeds are loaded and tests made before the first is used
              PixelSeed<C> sd[2];
              float dy[2], wv[2], z2sq[2], q[2];
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                sd[i] = sp[(kTile << lr) * i];
                dy[i] = (UNIT ? h : h * inv_s) - r[1];
                h += hstep;
                wv[i] = dy[i] - tt;
                const float z2 = wv[i] * r[4];
                z2sq[i] = z2 * z2;
                q[i] = zz1 + z2sq[i];
              }
              sp += (2 * kTile) << lr;
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                if (q[i] <= r2 && !(second_look && sd[i].hole())) {
                  const float ek = __builtin_amdgcn_exp2f(__builtin_fmaf(q[i], -0.5f * kLog2e, r[5]));
                  const float ed = ek * dy[i];
                  float Gs = -sd[i].gy;  // G / D
#pragma unroll
                  for (int c = 0; c < C; ++c) {
                    float m = mx[c];
                    if (ORDER == 1) m = __builtin_fmaf(r[kRecExpert + 2 * C + c], dy[i], m);
                    Gs = __builtin_fmaf(sd[i].g[c], m, Gs);
                    A[c] = __builtin_fmaf(sd[i].g[c], ek, A[c]);
                    if (ORDER == 1) Y[c] = __builtin_fmaf(sd[i].g[c], ed, Y[c]);
                  }
                  const float Hh = ek * Gs;  // H = w G
                  V = __builtin_fmaf(Hh, wv[i], V);
                  S2 = __builtin_fmaf(Hh, z2sq[i], S2);
                  R += Hh;
                }
              }
            }
          }
        };
        if (careful) {
          walk(std::true_type{});
          if (R == 0.0f && V == 0.0f && S2 == 0.0f) {  // nothing for z1 and the reciprocals to scale
            z1 = 0.0f;
            r[2] = r[4] = r[6] = 0.0f;
          }
        } else {
          walk(std::false_type{});
        }
        const float B2 = -V * r[4];
        const float B1 = -__builtin_fmaf(r[6], B2, z1 * R);
        float acc[16];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          acc[6 + c] = A[c];
          if (ORDER == 1) {
            acc[6 + C + c] = A[c] * dx;
            acc[6 + 2 * C + c] = Y[c];
          }
        }
        acc[0] = -B1 * r[2];
        acc[1] = -B2 * r[4];
        acc[2] = -B1 * z1;
        acc[3] = -B2 * z1 * r[4];
        acc[4] = S2;
        acc[5] = R;
#pragma unroll
        for (int i = 6 + C * (1 + 2 * ORDER); i < 16; ++i) acc[i] = 0.0f;
        tot = row_reduce16_masked(acc);
        if (careful || !__any(tot != tot)) break;
      }
      if (g + sub < n && l16 < PS) pair_grads[(size_t)out.y * PS + l16] = tot;
    }
  }
}

}  // namespace smoe
