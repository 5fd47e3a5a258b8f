// Fit-step kernels on gfx950 (Sec. VI-B: gradient descent with Adam on all kernel
// parameters, the centre learning rate decaying exponentially).
//
// A fit step runs three kernels (a fit's first step computes the render records first): the
// scatter of the (block, kernel) pairs into fixed-width block buckets, over each kernel's
// block rectangle computed from its model row (binning.hip), then
//   k_fit_tile: one wave (four on small rasters) per 16x16 block orders the block's bucket, renders the block
//     (image, D, squared error) and runs the backward over the same list while the
//     pixels' y, D and dL/dy are still in its registers -- the backward of a block needs
//     only that block's pixels, so nothing round-trips through HBM between the two;
//   k_adam_fit: per kernel, the sum of its block partials, Adam, re-materialization, and
//     the next step's render record.
// Cross-workgroup handoffs happen only at kernel boundaries: the 8 XCD L2 caches are not
// coherent with each other, so a device-scope fence per workgroup would cost more than a
// launch.  The step counter is read by every Adam workgroup and advanced by one: the
// scatter (the step's first kernel) copies it into a shadow status word that the later
// kernels read, so the single writer never races the readers.  A bucket overflow sets the
// step's flag (status word kStepFlags + parity of the step counter); Adam clears the next
// step's flag, which no kernel of this step reads.
#include "tile_math.h"

namespace smoe {
namespace {

struct FitTileArgs {
  Segs S;
  int shift;  // bucket entries: kernel id << shift | row of the entry's partial
  const float* __restrict__ records;
  int2* __restrict__ ranges;
  uint32_t* __restrict__ vals;
  uint32_t* __restrict__ vals_alt;
  int32_t* __restrict__ cursors;
  int32_t* __restrict__ status;
  int width;
  const float* __restrict__ target;
  float* __restrict__ image;  // null: the step's render is not stored
  float* __restrict__ denom;
  float* __restrict__ tile_loss;
  float* __restrict__ pair_grads;
};

// WAVES waves per block (tile_math.h).  One-wave workgroups are held to 64 VGPRs, 8 waves per
// SIMD.
template <int C, int ORDER, bool RBF, int TRUNC, int WAVES>
__global__ __launch_bounds__(kWave * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES == 1 ? 8 : 4, 8)))
void k_fit_tile(FitTileArgs a) {
  constexpr int ROWS = kStrips / WAVES;
  constexpr int LDS_FLOATS = kChunk * record_stride(C, ORDER);
  static_assert(LDS_FLOATS >= kRankList, "the ranking's scratch lives in the record buffer");
  // The forward's records and the backward's pixel seeds: the one after the other in the same
  // place, so that eight one-wave blocks fit a SIMD's share of LDS; side by side with several
  // waves to a block, where the backward then reads its records from LDS.  (Before both, a
  // long bucket's sort.)
  using LongSort = LongSortScratch<WAVES, 8192, (LDS_FLOATS >= 1024 ? 1024 : 512)>;
  constexpr int REC_BYTES = LDS_FLOATS * 4, SEED_BYTES = kTilePixels * (int)sizeof(PixelSeed<C>);
  constexpr int SEED_AT = WAVES == 1 ? 0 : REC_BYTES;
  constexpr int LDS_BYTES =
      max_of(max_of(REC_BYTES, SEED_AT + SEED_BYTES), (int)sizeof(LongSort));
  __shared__ float4 srec[(LDS_BYTES + 15) / 16];
  __shared__ __align__(16) BackwardScratch sc;  // sc.ent: also the entries of the chunk being staged
  __shared__ float s_err[WAVES == 1 ? 1 : kTilePixels];
  const int tile = xcd_block(blockIdx.x, a.S.T);
  const int t0 = a.status[kStepShadow];
  const int wave = wave_index<WAVES>();
  // The bucket's fill count; the cursor is then reset for the next step's scatter (the store
  // depends on the loaded value, so it cannot overtake the load; with several waves one
  // thread loads it for all).
  int cnt;
  if (WAVES == 1) {
    cnt = a.cursors[tile];
    if (threadIdx.x == 0 && cnt >= 0) a.cursors[tile] = 0;
  } else {
    if (threadIdx.x == 0) {
      const int c = a.cursors[tile];
      sc.ent[0] = (uint32_t)c;
      if (c >= 0) a.cursors[tile] = 0;
    }
    __syncthreads();
    cnt = __builtin_amdgcn_readfirstlane((int)sc.ent[0]);
    __syncthreads();
  }
  if (a.status[kStepFlags + (t0 & 1)] != 0) {
    // Some bucket overflowed: nothing is rendered or updated this step.  The status words
    // report the storage a step needs (blocks x longest bucket).
    if (threadIdx.x == 0 && cnt > a.width) {
      atomicMax(&a.status[2], cnt);
      atomicMax(&a.status[0], (int)min((long long)cnt * a.S.T, (long long)INT32_MAX));
      a.status[1] = 1;
    }
    return;
  }
  const int2 rg = make_int2(tile * a.width, tile * a.width + cnt);
  if (threadIdx.x == 0) a.ranges[tile] = rg;  // the gradient gather reads the list back
  const SegGrid sg = seg_of_tile(a.S, tile);
  // MSE of this raster: dL/dy = 2 (y - t) / (W H C); its squared errors are stored already
  // divided by W H C, so that the sum over all blocks is the sum of the rasters' MSEs.
  const float inv_n2 = 2.0f / ((float)sg.W * (float)sg.H * (float)C);
  const float inv_n = 1.0f / ((float)sg.W * (float)sg.H * (float)C);
  const BlockBox bb = block_box(sg, tile - sg.tile_offset);
  // Order the bucket (the scatter appended in arbitrary order).  A list of one chunk: a lane per
  // entry ranks it in registers while its record is on its way from memory, and writes the
  // record to its place for the forward; the backward's layout is worked out from the same
  // record, by the second wave if there is one.  The ordered entries go back for Adam's gather,
  // once every wave has read them.
  const int lane = threadIdx.x & 63;
  const int n = __builtin_amdgcn_readfirstlane(cnt);
  const bool one_chunk = n <= kChunk;
  if (one_chunk) {
    constexpr int RS = record_stride(C, ORDER), Q = RS / 4;
    uint32_t e = 0xFFFFFFFFu;
    int rank = 0;
    if (n > 0 && wave < 2) {
      float r[RS] = {};
      if (lane < n) {
        e = a.vals[rg.x + lane];
        load_record<RS>(r, reinterpret_cast<const float4*>(a.records + (size_t)(e >> a.shift) * RS));
      }
      rank = rank64(e, n, WAVES > 1 && wave == 0 ? reinterpret_cast<uint32_t*>(srec)
                                                 : reinterpret_cast<uint32_t*>(sc.out));
      if (wave == 0 && lane < n) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
          srec[rank * Q + q] = make_float4(r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]);
      }
      if (wave == (WAVES > 1 ? 1 : 0))
        lay_out_entries(bb, a.S.r, n, make_float4(r[0], r[1], r[2], r[3]), r[4], WAVES > 1 ? (uint32_t)rank : e >> a.shift,
                        partial_row(e, a.shift, true, 0, a.S.K, rg.x), sc);
    }
    __syncthreads();
    if (wave == 0 && lane < n) a.vals[rg.x + rank] = e;
  } else if (n <= kRankList) {
    rank_list<kWave * WAVES>(a.vals + rg.x, a.vals + rg.x, n, reinterpret_cast<uint32_t*>(srec),
                             (int)threadIdx.x, [] {
                               __threadfence_block();
                               __syncthreads();
                             });
  } else {
    sort_long(a.vals + rg.x, a.vals_alt + rg.x, n, a.shift, *reinterpret_cast<LongSort*>(srec));
  }

  const PixelCoords<ROWS> px = lane_pixels<WAVES>(sg, tile - sg.tile_offset);
  const BlockPixels bp = block_pixels<WAVES>(sg, tile - sg.tile_offset);
  const PixelValue<C>* tgt = reinterpret_cast<const PixelValue<C>*>(a.target) + bp.base;
  bool in[ROWS];
  PixelValue<C> t[ROWS], y[ROWS];
  auto load_target = [&]() {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      in[i] = in_raster(px.u, px.v0 + 4 * i, sg);
      if (in[i]) t[i] = tgt[bp.off + i * bp.step];
    }
  };
  if (WAVES > 1) load_target();  // on its way while the forward runs
  float D[ROWS], N[ROWS][C];
  forward_accumulate<C, ORDER, TRUNC, WAVES>(px, bb, a.S.r2, a.S.cut_scale, a.S.cut_offset,
                                             a.records, a.vals, a.shift, rg, srec, D, N, sc.ent,
                                             one_chunk);

  PixelSeed<C>* seeds = reinterpret_cast<PixelSeed<C>*>(reinterpret_cast<char*>(srec) + SEED_AT);
  if (WAVES == 1) {
    __syncthreads();  // the records are read: their place takes the seeds
    load_target();
  }
  float err[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    err[i] = 0.0f;
    PixelSeed<C> sd = hole_seed<C>();
    const bool cov = in[i] && D[i] > 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) y[i].v[c] = 0.0f;
    if (in[i]) {
      // 1/D by v_rcp_f32 (1 ulp); y = N / D refined from it, as in the render
      const float invD = RBF ? 1.0f : (cov ? __builtin_amdgcn_rcpf(D[i]) : 0.0f);
      float gy = 0.0f;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        // Eq. (2)-(4): y = N / D; Eq. (1): y = N
        const float yc = RBF ? N[i][c] : (cov ? div_refined(N[i][c], D[i], invD) : 0.0f);
        y[i].v[c] = yc;
        const float d = yc - t[i].v[c];
        err[i] = __builtin_fmaf(d, d, err[i]);
        if (cov) {
          const float g = d * inv_n2;
          if (!RBF) gy = __builtin_fmaf(g, yc, gy);
          sd.g[c] = g * invD;
        }
      }
      if (cov) sd.gy = live_gy(gy * invD);
    }
    seeds[((lane >> 4) + 4 * (i + ROWS * wave)) * kTile + (lane & 15)] = sd;
  }
  if (a.image) {
    PixelValue<C>* img = reinterpret_cast<PixelValue<C>*>(a.image) + bp.base;
    float* den = a.denom + bp.base;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      if (in[i]) {
        img[bp.off + i * bp.step] = y[i];
        den[bp.off + i * bp.step] = D[i];
      }
    }
  }
  const float sum = block_error<WAVES>(err, s_err);
  if (threadIdx.x == 0) a.tile_loss[tile] = sum * inv_n;

  // each partial row goes to the row its entry names, where Adam reads it
  const float2 o = block_base(sg, tile - sg.tile_offset);
  backward_accumulate<C, ORDER, true, WAVES>(bb, o.x, o.y, 1.0f, a.S.r, a.S.r2, a.records, a.vals,
                                             a.shift, true, rg, seeds, sc, one_chunk,
                                             WAVES > 1 && one_chunk ? srec : nullptr,
                                             a.pair_grads, a.S.K);
}

struct AdamFitArgs {
  Segs S;
  int shift;  // bucket entries: kernel id << shift | row of the partial (k_scatter_fixed)
  const int4* __restrict__ tile_rects;  // the step's block rectangles (from its scatter)
  const int2* __restrict__ ranges;
  const uint32_t* __restrict__ vals;
  const float* __restrict__ pair_grads;
  const float* __restrict__ tile_loss;  // per-block squared errors / (W H C)
  int32_t* __restrict__ status;
  StepScalarsArgs step;
  float* __restrict__ raw;
  float* __restrict__ m;
  float* __restrict__ v;
  float* __restrict__ model;
  float* __restrict__ grads;
  float* __restrict__ records;
};


// Fit-step Adam fused with the re-materialization.  16 lanes per kernel: lane i owns raw
// parameter i -- its gradient (the sum of the kernel's block partials), Adam with the group's
// learning rate, the re-materialized value -- and writes field i of the new render record
// (the next step's scatter derives the block rectangle from the new model row).  Block 0
// also reduces the per-block squared errors into the loss.  After an overflow the
// parameters stay as they are, and the records are rewritten from them unchanged.
constexpr int kAdamThreads = 256;
// (held to 64 VGPRs: 8 waves per SIMD to overlap the gather's loads)
template <int C, int ORDER>
__global__ __launch_bounds__(kAdamThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
void k_adam_fit(AdamFitArgs f) {
  constexpr int NP = num_params(C, ORDER);
  constexpr int NE = expert_floats(C, ORDER);
  constexpr int RS = record_stride(C, ORDER);
  __shared__ float s_red[kAdamThreads / 64];
  const smoe_adam_config& ad = f.step.adam;
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = gid >> 4, i = gid & 15;
  const bool live = j < f.S.K;
  const size_t e = (size_t)j * NP + i;
  // Every load that depends on no other is issued before the first wait: the status words
  // (the completed steps, copied by this step's scatter, and both overflow flags), the step's
  // Adam scalars (written by the scatter), the kernel's block rectangle and Adam's state.
  const int t0 = f.status[kStepShadow];
  const int flag0 = f.status[kStepFlags], flag1 = f.status[kStepFlags + 1];
  const float lr_mu = f.step.scalars[0], bc1 = f.step.scalars[1], bc2 = f.step.scalars[2];
  int4 rc = make_int4(0, 0, -1, -1);
  float m0 = 0.0f, v0 = 0.0f, raw0 = 0.0f;
  if (live) {
    rc = f.tile_rects[j];
    if (i < NP) {
      m0 = f.m[e];
      v0 = f.v[e];
      raw0 = f.raw[e];
    }
  }
  const bool skip = ((t0 & 1) ? flag1 : flag0) != 0;
  if (blockIdx.x == 0 && !skip) {
    // Loss: the whole workgroup sums the per-block squared errors in a fixed order, four
    // independent float4 streams per thread so that the loads overlap.
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const int T4 = f.S.T >> 2;
    const float4* tl4 = reinterpret_cast<const float4*>(f.tile_loss);
    for (int q = threadIdx.x; q < T4; q += 4 * kAdamThreads) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int qq = q + u * kAdamThreads;
        if (qq < T4) {
          const float4 v = tl4[qq];
          acc[u] += (v.x + v.y) + (v.z + v.w);
        }
      }
    }
    for (int t = (T4 << 2) + threadIdx.x; t < f.S.T; t += kAdamThreads) acc[0] += f.tile_loss[t];
    float tot = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
      float sum = 0.0f;
      for (int w = 0; w < kAdamThreads / 64; ++w) sum += s_red[w];
      const float loss = sum;
      if (f.step.loss_out) f.step.loss_out[0] = loss;
      if (f.step.loss_history && t0 < f.step.max_steps) f.step.loss_history[t0] = loss;
    }
  }

  float pm = 0.0f;  // materialized value of parameter i after the step
  if (live && skip && i < NP) pm = f.model[e];
  const bool upd = live && !skip && i < NP;
  // Every lane takes part in the gather's row reduction and the finishing shuffles; the
  // expert slopes are those of the raw row (the render record this step used holds the same
  // numbers).
  const float gi = finish_gradient<C, ORDER, 6>(
      gather_param_fit<NP>(j, live && !skip, f.S, rc, f.ranges, f.vals, f.pair_grads, f.shift),
      live && !skip, raw0);
  if (upd) {
    const float lr = i < 2 ? lr_mu : (i < 5 ? ad.lr_chol : (i == 5 ? ad.lr_rho : ad.lr_expert));
    const float mi = ad.beta1 * m0 + (1.0f - ad.beta1) * gi;
    const float vi = ad.beta2 * v0 + (1.0f - ad.beta2) * gi * gi;
    f.m[e] = mi;
    f.v[e] = vi;
    const float p = raw0 - lr * (mi / bc1) / (sqrtf(vi / bc2) + ad.eps);
    f.raw[e] = p;
    pm = (i == 2 || i == 4) ? expf(p) : p;
    f.model[e] = pm;
    if (f.grads) f.grads[e] = gi;
  }
  // The kernel's new row, shared inside its group of 16 lanes.
  const float mux = __shfl(pm, 0, 16), muy = __shfl(pm, 1, 16), l11 = __shfl(pm, 2, 16);
  const float l21 = __shfl(pm, 3, 16), l22 = __shfl(pm, 4, 16), rho = __shfl(pm, 5, 16);
  const float prev = __shfl_up(pm, 1, 16);  // parameter i - 1
  // A row with a NaN or infinite parameter covers no block in the next step (it takes part
  // nowhere) and sets the non-finite status word.
  const unsigned long long nf = __ballot(i < NP && !__builtin_isfinite(pm));
  const bool row_nonfinite = ((nf >> (threadIdx.x & 48)) & 0xFFFFull) != 0;
  if (live) {
    if (i < RS) {
      const float i22 = 1.0f / l22;
      float fld;
      if (i == 0) fld = mux;
      else if (i == 1) fld = muy;
      else if (i == 2) fld = 1.0f / l11;
      else if (i == 3) fld = l21;
      else if (i == 4) fld = i22;
      else if (i == 5) fld = rho * kLog2e;
      else if (i == 6) fld = l21 * i22;
      else if (i < kRecExpert + NE) fld = prev;
      else fld = 0.0f;
      f.records[(size_t)j * RS + i] = fld;
    }
    if (i == 0 && row_nonfinite) f.status[kNonfinite] = 1;
  }
  // The counter itself is written once; every workgroup read the shadow copy instead.  The
  // next step's overflow flag is cleared here: no kernel of this step reads it.
  if (blockIdx.x == 0 && threadIdx.x == 0 && !skip) {
    f.step.step[0] = t0 + 1;
    f.status[kStepFlags + ((t0 + 1) & 1)] = 0;
  }
}

// Reporting: the loss of each raster of the last fit step (one workgroup per segment sums
// its blocks' normalised squared errors in a fixed order).
__global__ __launch_bounds__(256) void k_segment_losses(Segs S, const float* __restrict__ tile_loss,
                                                        float* __restrict__ out) {
  __shared__ float s_red[4];
  const smoe_segment seg = S.tab ? S.tab[blockIdx.x] : S.one;
  const int T0 = seg.tile_offset;
  const int Ts = blocks_across(seg.width, seg.origin_x) * blocks_across(seg.height, seg.origin_y);
  float acc = 0.0f;
  for (int t = threadIdx.x; t < Ts; t += 256) acc += tile_loss[T0 + t];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}

__global__ __launch_bounds__(128) void k_materialize(int n_rows, int NP,
                                                     const float* __restrict__ raw,
                                                     float* __restrict__ model) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rows * NP) return;
  const int k = i % NP;
  const float x = raw[i];
  model[i] = (k == 2 || k == 4) ? expf(x) : x;
}

}  // namespace

hipError_t launch_fit_tile(const smoe_fit_state& st, const Segs& S, int width, int shift,
                           const float* target, hipStream_t s) {
  const smoe_bins& b = st.bins;
  FitTileArgs a{S,        shift,     b.records, reinterpret_cast<int2*>(b.ranges),
                b.vals,   b.vals_alt, b.tile_counts, b.status, width,
                target,   st.write_render ? st.image : nullptr,
                st.write_render ? st.denom : nullptr,
                b.tile_loss, b.pair_grads};
  with_shape(st.C, st.order, S, [&](auto sh) {
    using T = decltype(sh);
    if (split_blocks(S))
      k_fit_tile<T::C, T::ORDER, T::RBF, T::TRUNC, 4><<<S.T, 4 * kWave, 0, s>>>(a);
    else
      k_fit_tile<T::C, T::ORDER, T::RBF, T::TRUNC, 1><<<S.T, kWave, 0, s>>>(a);
  });
  return hipGetLastError();
}

hipError_t launch_adam_fit(const smoe_fit_state& st, const Segs& S, int shift, float* loss_out,
                           hipStream_t s) {
  const smoe_bins& b = st.bins;
  AdamFitArgs f{S,
                shift,
                reinterpret_cast<const int4*>(b.tile_rects),
                reinterpret_cast<const int2*>(b.ranges),
                b.vals,
                b.pair_grads,
                b.tile_loss,
                b.status,
                make_step_scalars_args(st, loss_out),
                st.raw,
                st.adam_m,
                st.adam_v,
                st.model,
                st.grads,
                b.records};
  // at least one workgroup, so that the loss and the step counter advance even for K = 0
  const int blocks = max(1, (int)(((long long)S.K * 16 + kAdamThreads - 1) / kAdamThreads));
  if (st.C == 1 && st.order == 0) k_adam_fit<1, 0><<<blocks, kAdamThreads, 0, s>>>(f);
  else if (st.C == 1 && st.order == 1) k_adam_fit<1, 1><<<blocks, kAdamThreads, 0, s>>>(f);
  else if (st.C == 3 && st.order == 0) k_adam_fit<3, 0><<<blocks, kAdamThreads, 0, s>>>(f);
  else k_adam_fit<3, 1><<<blocks, kAdamThreads, 0, s>>>(f);
  return hipGetLastError();
}

hipError_t launch_segment_losses(const Segs& S, const smoe_bins& b, float* out, hipStream_t s) {
  k_segment_losses<<<S.tab ? S.n : 1, 256, 0, s>>>(S, b.tile_loss, out);
  return hipGetLastError();
}

hipError_t launch_materialize(int K, int C, int order, const float* raw, float* model,
                              hipStream_t s) {
  const int NP = num_params(C, order);
  const long long n = (long long)K * NP;
  if (n == 0) return hipSuccess;
  k_materialize<<<(int)((n + 127) / 128), 128, 0, s>>>(K, NP, raw, model);
  return hipGetLastError();
}

}  // namespace smoe
