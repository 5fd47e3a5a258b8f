// Device building blocks shared by the standalone binning calls and the fused fit step:
// the kernel box (Sec. IV-B), the render record and the ordering of a block's list by kernel id
// (Sec. IV-C).  Internal header.
#pragma once

#include "smoe_internal.h"

namespace smoe {

constexpr int kStepShadow = 4;  // status word: completed steps, copied by the step's first kernel
constexpr int kStepFlags = 5;   // status words 5, 6: the fit step's overflow flag by step parity
constexpr int kNonfinite = 7;   // status word: a kernel row with a NaN or infinite parameter was
                                // seen (cleared by each binning's first kernel and at the start
                                // of a fit; sticky over a fit's steps)
constexpr int kNonfiniteOut = 3;  // status word: the binning's copy of kNonfinite

// Native 16x16 block index of a native coordinate, floor(x / 16) (x * 2^-4 is exact).
__host__ __device__ __forceinline__ float native_block(float x) { return floorf(x * 0.0625f); }

// Output-block range [t0, t1] of one axis of a raster (n points sampled at
// ((o + u) + 0.5) * inv_s; blocks aligned to multiples of 16 in o + u) holding a point whose
// native block lies in [b0, b1], and the
// native range clamped to the blocks the raster's points reach.  Native block b is the 16
// scale output pixels from o + u = 16 scale b on -- the binary32 sample coordinates included,
// over the whole accepted range -- so both ends are had directly.  (A binary search over the
// sample coordinates gives the same: 48 dependent steps per kernel at scale 4, 4096^2.)
// False when no point is in [b0, b1] (or NaN).
__host__ __device__ __forceinline__ bool output_axis(float b0, float b1, int n, int o, int scale,
                                                     float inv_s, int& t0, int& t1, int& nb0,
                                                     int& nb1) {
  const float first = native_block(sample_coord(0, o, inv_s));
  const float last = native_block(sample_coord(n - 1, o, inv_s));
  if (!(b1 >= first) || !(b0 <= last)) return false;
  nb0 = (int)fmaxf(b0, first);
  nb1 = (int)fminf(b1, last);
  const int u0 = max(0, 16 * scale * nb0 - o);
  const int u1 = min(n - 1, 16 * scale * (nb1 + 1) - 1 - o);
  // blocks of the grid aligned to multiples of 16 in o + u, numbered from the raster's first
  t0 = first_block(o + u0) - first_block(o);
  t1 = first_block(o + u1) - first_block(o);
  return true;
}

// A kernel's blocks on one raster: `tile` = its output-block rectangle (tx0, ty0, tx1, ty1)
// and `native` = its native 16x16 blocks (bx0, by0, bx1, by1) clamped to those the raster's
// points reach; both (0, 0, -1, -1) when empty.
struct KernelRects {
  int4 tile, native;
};

// The blocks of one kernel: the native blocks its square box of half-side
// R = r sqrt(lambda_max(L L^T)) around mu covers -- with the block lists deciding the render
// (SMOE_TRUNC_GRADIENT) those holding a native pixel centre inside the box, with the ellipse
// deciding (SMOE_TRUNC_RENDER) those the box overlaps, so that every point inside the ellipse
// is a member at any scale -- or those of its tight axis-aligned box of the
// ellipse's x and y extents (widened by a rounding margin, capped at R) -- as the exact
// binary32 sequences of the ABI contract; the raster's output blocks are those holding a
// sample point in them.
__device__ __forceinline__ KernelRects kernel_rects(float mux, float muy, float l11, float l21,
                                                    float l22, const SegGrid& g, float r, int box,
                                                    int trunc) {
  const float sxx = l11 * l11;
  const float sxy = l11 * l21;
  const float syy = l21 * l21 + l22 * l22;
  const float h = 0.5f * (sxx + syy);
  const float d = 0.5f * (sxx - syy);
  const float lam = h + sqrtf(d * d + sxy * sxy);
  const float R = r * sqrtf(lam);
  float Rx = R, Ry = R;
  if (box == SMOE_BOX_TIGHT) {
    const float m = (fabsf(mux) + fabsf(muy) + R) * 0x1p-18f;
    Rx = fminf(R, r * fabsf(l11) * 1.0009765625f + m);
    Ry = fminf(R, r * sqrtf(syy) * 1.0009765625f + m);
  }
  float bx0f, bx1f, by0f, by1f;
  if (trunc == SMOE_TRUNC_GRADIENT) {
    // the blocks of the native pixel centres c + 0.5 inside the box: c from ceil(lo - 0.5)
    // to floor(hi - 0.5) (empty if none)
    const float cx0 = ceilf((mux - Rx) - 0.5f), cx1 = floorf((mux + Rx) - 0.5f);
    const float cy0 = ceilf((muy - Ry) - 0.5f), cy1 = floorf((muy + Ry) - 0.5f);
    bx0f = cx0 <= cx1 ? native_block(cx0) : 1.0f;
    bx1f = cx0 <= cx1 ? native_block(cx1) : 0.0f;
    by0f = cy0 <= cy1 ? native_block(cy0) : 1.0f;
    by1f = cy0 <= cy1 ? native_block(cy1) : 0.0f;
  } else {
    // the blocks the box overlaps: floor(lo/16) .. ceil(hi/16) - 1
    bx0f = native_block(mux - Rx);
    bx1f = ceilf((mux + Rx) * 0.0625f) - 1.0f;
    by0f = native_block(muy - Ry);
    by1f = ceilf((muy + Ry) * 0.0625f) - 1.0f;
  }
  KernelRects k;
  k.tile = make_int4(0, 0, -1, -1);
  k.native = make_int4(0, 0, -1, -1);
  if (!(bx0f <= bx1f) || !(by0f <= by1f)) return k;
  int tx0, tx1, ty0, ty1, bx0, bx1, by0, by1;
  if (output_axis(bx0f, bx1f, g.W, g.ox, g.scale, g.inv_s, tx0, tx1, bx0, bx1) &&
      output_axis(by0f, by1f, g.H, g.oy, g.scale, g.inv_s, ty0, ty1, by0, by1)) {
    k.tile = make_int4(tx0, ty0, tx1, ty1);
    k.native = make_int4(bx0, by0, bx1, by1);
  }
  return k;
}

// n / d from r = v_rcp_f32(d) (within 1 ulp of 1/d) and one Newton-Raphson correction of
// the quotient: q = n r, q + r (n - d q).  Within an ulp of the correctly rounded quotient
// (equal to it in all but about 5 of 10^7 random cases), and exactly 1 when n == d, so the
// gates still sum to one bit for bit; a few instructions instead of the scaled IEEE
// division sequence.
__device__ __forceinline__ float div_refined(float n, float d, float r) {
  const float q = n * r;
  return __builtin_fmaf(__builtin_fmaf(-d, q, n), r, q);
}

__device__ __forceinline__ int rect_count(int4 rc) {
  return rc.z < rc.x ? 0 : (rc.z - rc.x + 1) * (rc.w - rc.y + 1);
}

// Float4 number `quad` of the render record of a kernel row from its materialized parameter
// row p (layout in smoe_internal.h; the record is 16-byte aligned): field f holds, beyond the
// seven geometry fields, expert float f - 7 = p[f - 1], and zero padding after the experts.
// (l11, l21, l22): the Cholesky factor the record is built for (the row's own, or divided by
// a sharpening factor).
__device__ __forceinline__ void write_record_quad(float* __restrict__ rec,
                                                  const float* __restrict__ p, int ne, int quad,
                                                  float l11, float l21, float l22) {
  float4* r4 = reinterpret_cast<float4*>(rec);
  if (quad == 0) {
    r4[0] = make_float4(p[0], p[1], 1.0f / l11, l21);
  } else if (quad == 1) {
    const float i22 = 1.0f / l22;
    r4[1] = make_float4(i22, p[5] * kLog2e, l21 * i22, ne > 0 ? p[6] : 0.0f);
  } else {
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int f = 4 * quad + k;
      v[k] = f < kRecExpert + ne ? p[f - 1] : 0.0f;
    }
    r4[quad] = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// Orders this wave's LDS and memory accesses before it against those after it, as seen by
// its own lanes (a wave's LDS accesses execute in program order: the compiler must keep it).
// Unlike a workgroup barrier it may be used by one wave of several.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The rank of a lane's entry e among the n <= 64 distinct ones of a wave (e of lanes 0 .. n - 1;
// the others pass 0xFFFFFFFF): the number of entries below it, from broadcast reads of all of
// them in LDS.  scratch: 64 u32 of LDS, 16-byte aligned.
__device__ __forceinline__ int rank64(uint32_t e, int n, uint32_t* __restrict__ scratch) {
  scratch[threadIdx.x & 63] = e;
  wave_sync();
  int rank = 0;
  const uint4* s4 = reinterpret_cast<const uint4*>(scratch);
  for (int j = 0; j < (n + 3) >> 2; ++j) {
    const uint4 q = s4[j];
    rank += (q.x < e ? 1 : 0) + (q.y < e ? 1 : 0) + (q.z < e ? 1 : 0) + (q.w < e ? 1 : 0);
  }
  wave_sync();
  return rank;
}

// Orders a list of n <= kRankList distinct entries from[0, n) into to[0, n) (which may be from) with NT
// threads, of which the caller is number tid: an entry's place is the number of entries below it,
// counted as in rank64.  lds: kRankList u32, 16-byte aligned; sync: a barrier of the NT threads.
// A bitmap of the ids (sort_long) costs a workgroup about 1.7 us a window whatever n is: binning of
// 262144 kernels at 2048^2 (lists of about 105) with bitmaps from 65 entries on 133 us, and 237 if
// the kernels are in random order (eight windows); with this up to 128 / 192 / 256 entries 124 / 121 /
// 121 and 136 / 119 / 119, but lists of up to 518 at scale 3 102 / 102 / 108.
constexpr int kRankList = 192;
template <int NT, class Sync>
__device__ __forceinline__ void rank_list(const uint32_t* from, uint32_t* to, int n,
                                          uint32_t* __restrict__ lds, int tid, Sync&& sync) {
  for (int i = tid; i < ((n + 3) & ~3); i += NT) lds[i] = i < n ? from[i] : 0xFFFFFFFFu;
  sync();
  const uint4* l4 = reinterpret_cast<const uint4*>(lds);
  for (int i = tid; i < n; i += NT) {
    const uint32_t e = lds[i];
    int rank = 0;
    for (int j = 0; j < (n + 3) >> 2; ++j) {
      const uint4 q = l4[j];
      rank += (q.x < e ? 1 : 0) + (q.y < e ? 1 : 0) + (q.z < e ? 1 : 0) + (q.w < e ? 1 : 0);
    }
    to[rank] = e;
  }
  sync();
}

// Scratch of sort_long: a bitmap over a window of kernel ids and, per word, the ids below it; or a
// run of entries.
template <int WAVES, int WINDOW_, int RUN_>
struct LongSortScratch {
  static constexpr int WINDOW = WINDOW_, RUN = RUN_;
  union {
    struct {
      uint32_t bits[WINDOW / 32];
      uint32_t below[WINDOW / 32];
    };
    uint32_t run[RUN];
  };
  uint32_t wave[WAVES], lo[WAVES], hi[WAVES];
};

// Orders distinct entries seg[0, n) ascending with NT threads, through alt[0, n): a bitonic sort of
// each run of RUN entries in LDS, then merges of pairs of runs, in which an entry's place is its
// index in its own run plus the number of smaller entries in the other.
template <int NT, int RUN>
__device__ __forceinline__ void sort_runs(uint32_t* seg, uint32_t* alt, int n,
                                          uint32_t* __restrict__ run) {
  const int tid = threadIdx.x;
  for (int c0 = 0; c0 < n; c0 += RUN) {
    const int m = min(RUN, n - c0);
    int p2 = 2;
    while (p2 < m) p2 <<= 1;
    for (int i = tid; i < p2; i += NT) run[i] = i < m ? seg[c0 + i] : 0xFFFFFFFFu;
    __syncthreads();
    for (int k = 2; k <= p2; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < p2 >> 1; i += NT) {
          const int a = 2 * i - (i & (j - 1)), b = a + j;
          const uint32_t x = run[a], y = run[b];
          if ((x > y) == ((a & k) == 0)) {
            run[a] = y;
            run[b] = x;
          }
        }
        __syncthreads();
      }
    }
    for (int i = tid; i < m; i += NT) seg[c0 + i] = run[i];
    __threadfence_block();
    __syncthreads();
  }
  uint32_t *src = seg, *dst = alt;
  for (int width = RUN; width < n; width <<= 1) {
    for (int i = tid; i < n; i += NT) {
      const int own = i / width * width;               // begin of the entry's run
      const bool left = (own / width & 1) == 0;
      const int other = left ? own + width : own - width;
      const uint32_t v = src[i];
      int lo = min(other, n), hi = min(other + width, n);
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (src[mid] < v) lo = mid + 1;
        else hi = mid;
      }
      dst[min(own, other) + (i - own) + (lo - min(other, n))] = v;
    }
    __threadfence_block();
    __syncthreads();
    uint32_t* t = src;
    src = dst;
    dst = t;
  }
  if (src != seg) {
    for (int i = tid; i < n; i += NT) seg[i] = src[i];
    __threadfence_block();
    __syncthreads();
  }
}

// Orders a list of n > kRankList entries seg[0, n) by kernel id (entry >> shift; the ids are
// distinct) with a workgroup of WAVES waves, through alt[0, n).  Where the list's ids lie close
// together, as they do in a model whose kernels' order follows the image, an entry's place is the
// number of ids below its own, which a bitmap of the ids present gives -- one pass to set the bits,
// one over the words for the running counts, one to place the entries -- for every window of
// WINDOW ids between the list's least and greatest.  The work is proportional to n plus
// the ids' span / 32, against n log^2 n for a sorting network by one wave, which took 97 us over
// 1024 lists of 500 to 900 ids; this takes 18 us.  Ids spread over more than kRunWindows windows, in
// a list that fits a run, go by sort_runs (a million kernels in random order at 2048^2, lists of up
// to 360: binning 810 -> 437 us, fit step 1580 -> 1096; at four windows bitmaps take 117 us where
// runs take 131, at twelve 197 against 160).  Lists longer than a run do from kMergeWindows on:
// bitmaps against merged runs, lists of about 2400 over 18 windows 973 / 984 us, of 6900 over 40
// 3243 / 2832, of 5700 over 122 5532 / 2820.
// All threads of the workgroup call it, with the same arguments; the result is in seg.
constexpr uint32_t kRunWindows = 4, kMergeWindows = 24;
template <int WAVES, int WINDOW, int RUN>
__device__ __forceinline__ void sort_long(uint32_t* __restrict__ seg, uint32_t* __restrict__ alt, int n,
                                          int shift, LongSortScratch<WAVES, WINDOW, RUN>& sc) {
  constexpr int NT = 64 * WAVES, WORDS = WINDOW / 32, PER = WORDS / NT;
  static_assert(WORDS % NT == 0, "whole words per thread");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t lo = 0xFFFFFFFFu, hi = 0;
  for (int i = tid; i < n; i += NT) {
    const uint32_t id = seg[i] >> shift;
    lo = min(lo, id);
    hi = max(hi, id);
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
  }
  if (lane == 0) {
    sc.lo[wave] = lo;
    sc.hi[wave] = hi;
  }
  __syncthreads();
  for (int w = 0; w < WAVES; ++w) {
    lo = min(lo, sc.lo[w]);
    hi = max(hi, sc.hi[w]);
  }
  const uint32_t windows = (hi - lo) / WINDOW + 1;
  if (windows > (n <= RUN ? kRunWindows : kMergeWindows)) {
    sort_runs<NT, RUN>(seg, alt, n, sc.run);
    return;
  }
  uint32_t done = 0;  // entries of the windows before
  for (uint32_t base = lo; base <= hi; base += WINDOW) {
    for (int i = tid; i < WORDS; i += NT) sc.bits[i] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
      const uint32_t d = (seg[i] >> shift) - base;
      if (d < (uint32_t)WINDOW) atomicOr(&sc.bits[d >> 5], 1u << (d & 31));
    }
    __syncthreads();
    uint32_t c[PER], mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      c[k] = mine;
      mine += __popc(sc.bits[tid * PER + k]);
    }
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = (uint32_t)__shfl_up((int)incl, off);
      if (lane >= off) incl += o;
    }
    if (lane == 63) sc.wave[wave] = incl;
    __syncthreads();
    uint32_t before = done + incl - mine, total = done;
    for (int w = 0; w < WAVES; ++w) {
      if (w < wave) before += sc.wave[w];
      total += sc.wave[w];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) sc.below[tid * PER + k] = before + c[k];
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
      const uint32_t e = seg[i], d = (e >> shift) - base;
      if (d < (uint32_t)WINDOW)
        alt[sc.below[d >> 5] + __popc(sc.bits[d >> 5] & ((1u << (d & 31)) - 1u))] = e;
    }
    done = total;
    __syncthreads();
  }
  for (int i = tid; i < n; i += NT) seg[i] = alt[i];
  __threadfence_block();
  __syncthreads();
}

// Arguments the fit step's Adam kernel needs to record the loss and advance the step.
struct StepScalarsArgs {
  int32_t* step;
  float* scalars;
  float* loss_out;
  float* loss_history;
  int max_steps;
  smoe_adam_config adam;
};

inline StepScalarsArgs make_step_scalars_args(const smoe_fit_state& st, float* loss_out) {
  return StepScalarsArgs{st.step, st.scalars, loss_out, st.loss_history, st.max_steps, st.adam};
}

// The per-step Adam scalars of step t0 (Sec. VI-B): out[0] = the centre learning rate,
// decaying exponentially from lr_mu to lr_mu_final over total_steps; out[1], out[2] = the bias
// corrections 1 - beta1^(t0+1), 1 - beta2^(t0+1).  Computed once per step by one thread.
__device__ __forceinline__ void adam_step_scalars(const smoe_adam_config& ad, int t0,
                                                  float* __restrict__ out) {
  float lr_mu = ad.lr_mu;
  if (ad.total_steps > 0 && ad.lr_mu > 0.0f && ad.lr_mu_final > 0.0f)
    lr_mu = ad.lr_mu * powf(ad.lr_mu_final / ad.lr_mu, (float)t0 / (float)ad.total_steps);
  out[0] = lr_mu;
  out[1] = 1.0f - powf(ad.beta1, (float)(t0 + 1));
  out[2] = 1.0f - powf(ad.beta2, (float)(t0 + 1));
}

}  // namespace smoe
