// Binning on gfx950: per-kernel box and render record, per-block counting, ordering of the
// (block, kernel) pairs and block ranges (Sec. IV-B "geometry shader", Sec. IV-C "subset
// kernel selection for each block").
//
// Ordering.  The pairs are ordered by block id and, within a block, by kernel id: the
// order a stable LSD radix sort by block id gives the kernel-major pair list.  It is
// computed as a radix sort whose single digit is the whole block id (2^14 buckets at
// 2048^2): an atomic histogram of the digit, one exclusive scan of the histogram (which
// is also the block ranges), a scatter into the buckets, and a per-bucket ranking of the
// kernel ids that restores the stable order the atomic scatter does not keep.
// Every pass is integer work over a few MB, so the design minimises launches, not bytes.
// The fit step uses fixed-width buckets instead (k_scatter_fixed): no histogram and no scan,
// the bucket of block t is entries [t W, t W + W) of the pair storage.
#include <type_traits>

#include "device_common.h"

namespace smoe {
namespace {

// Lanes per kernel row (LANES): a group of lanes shares the row's blocks, so that the atomics of
// one kernel run side by side.  In the kernels whose every lane also works out the row's
// rectangle (k_preprocess, k_scatter_fixed) sixteen pay while that work does not fill the chip.
// Measured, 4 / 16 / 64 lanes: fit scatter at 4096 rows 6.4 / 4.8 / 7.4 us, at 65536 rows 11.3 /
// 13.6 / 45.9; k_preprocess at 3024 rows 7.8 / 6.7 / 11.0, at 65536 rows 12.6 / 21.5 / 70, at 4000
// rows of 150 blocks each 57 / 37 / 38.  Rows of a few blocks have nothing to share out: four
// (few_blocks; k_scatter_fixed over 66564 rows of a block each 11.3 against 24.6).  k_scatter
// reads the rectangle: sixteen always (65536
// rows 9.6 / 9.5 / 36, a batch of serving requests 108 / 71 / 140, the 4000 wide rows 104 /
// 53 / 37).
constexpr int kScatterLanes = 16, kManyKernels = 16384;
// Calls f(std::integral_constant<int, LANES>) for the kernel rows of S.
template <class F>
inline void with_lanes(const Segs& S, F&& f) {
  if (S.K > kManyKernels || few_blocks(S)) f(std::integral_constant<int, 4>{});
  else f(std::integral_constant<int, 16>{});
}

// The kernel that group g of a binning kernel's lanes takes: every
// 8th of 128 consecutive kernel ids (a bijection on each complete run of 128; the ids past
// the last one keep their order).  Neighbouring ids are neighbours in the image (the grid
// initialisation's order, which the kernels keep as they move), so a wave's counter and
// cursor atomics stay within a few blocks; spreading them over eight times as many ids keeps
// that locality while fewer atomics of one instruction meet on the same counter, where they
// serialise.  Any order gives the same counts and, up to the order inside a bucket, which
// the sorts that follow remove, the same buckets.
__device__ __forceinline__ int binning_kernel(int g, int K) {
  return (g | 127) < K ? (g & ~127) + ((g & 15) << 3) + ((g >> 4) & 7) : g;
}

// Every lane of a kernel's group reads the row and computes the output-block and native-block
// rectangles; lane 0 writes them and the count, lane q the q-th float4 of the render record,
// and (tile_counts not null) lane q adds one to the counts of the kernel's covered blocks q, q +
// LANES, ... (row-major).  A row with a NaN or infinite parameter covers no block (it takes
// part nowhere) and sets the non-finite status word.
template <int LANES>
__global__ __launch_bounds__(256) void k_preprocess(int C, int order,
                                                    const float* __restrict__ params, Segs S,
                                                    int4* __restrict__ tile_rects,
                                                    int4* __restrict__ native_rects,
                                                    int32_t* __restrict__ counts,
                                                    float* __restrict__ records, int rs,
                                                    int32_t* __restrict__ tile_counts,
                                                    int32_t* __restrict__ status) {
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int g = gid / LANES, lq = gid % LANES;
  if (g >= S.K) return;
  const int j = binning_kernel(g, S.K);
  const SegGrid sg = seg_of_kernel(S, j);
  const int ne = expert_floats(C, order);
  const float* p = params + (size_t)(sg.param_offset + (j - sg.kernel_offset)) * (6 + ne);
  // native sharpening: the raster sees L / f (a correctly rounded binary32 division)
  float l11 = p[2], l21 = p[3], l22 = p[4];
  if (sg.sharpen != 1.0f) {
    l11 = l11 / sg.sharpen;
    l21 = l21 / sg.sharpen;
    l22 = l22 / sg.sharpen;
  }
  bool finite = __builtin_isfinite(l11) && __builtin_isfinite(l21) && __builtin_isfinite(l22);
  for (int k = 0; k < 6 + ne; ++k) finite = finite && __builtin_isfinite(p[k]);
  KernelRects kr;
  if (finite) {
    kr = kernel_rects(p[0], p[1], l11, l21, l22, sg, S.r, S.box, S.trunc);
  } else {
    kr.tile = kr.native = make_int4(0, 0, -1, -1);
  }
  const int4 rc = kr.tile;
  if (lq == 0) {
    tile_rects[j] = rc;
    native_rects[j] = kr.native;
    counts[j] = rect_count(rc);
    if (!finite) status[kNonfinite] = 1;
  }
  if (lq < rs / 4) write_record_quad(records + (size_t)j * rs, p, ne, lq, l11, l21, l22);
  if (tile_counts) count_blocks(rc, sg, tile_counts, lq, LANES);
}

// Exclusive scan of the per-block counts into [begin, end) ranges, with P, the overflow flag
// and the longest list into status.  A workgroup takes kScanChunk consecutive blocks, four
// counts a thread; no workgroup waits for another.  What lies before its chunk, and the total
// (on an overflow every range is written empty), each workgroup sums for itself: from all the
// counts (part null), or from the chunks' sums that k_scan_sums left in part.  Summing all
// the counts is quadratic in the number of chunks, so it serves up to kScanDirect blocks
// (4096^2 pixels: 256 KB read by each of 16 workgroups), where it saves a launch.  One
// workgroup that walked all chunks took 7.7 us at 16384 blocks and 107 us for the 220 000 of a
// batch of serving requests; the two kernels take 5.6 + 4.6 us there, the direct one 6.8 us at
// 16384 blocks.  The batch of twelve requests 1569 -> 1469 us.
constexpr int kScanThreads = 1024, kScanChunk = 4 * kScanThreads, kScanDirect = 65536;

// Sum and maximum over a chunk of counts (part of T), in every thread of the workgroup.
struct ChunkTotals {
  long long before, total;
  int longest;
};
__device__ __forceinline__ ChunkTotals workgroup_totals(ChunkTotals t) {
  __shared__ long long s_before[kScanThreads / 64], s_total[kScanThreads / 64];
  __shared__ int s_max[kScanThreads / 64];
  for (int off = 32; off > 0; off >>= 1) {
    t.before += __shfl_xor(t.before, off);
    t.total += __shfl_xor(t.total, off);
    t.longest = max(t.longest, __shfl_xor(t.longest, off));
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_before[wave] = t.before;
    s_total[wave] = t.total;
    s_max[wave] = t.longest;
  }
  __syncthreads();
  ChunkTotals r{0, 0, 0};
  for (int w = 0; w < kScanThreads / 64; ++w) {
    r.before += s_before[w];
    r.total += s_total[w];
    r.longest = max(r.longest, s_max[w]);
  }
  return r;
}

// Counts q .. q + 3 (zero past T; the array is 16-byte aligned).
__device__ __forceinline__ int4 four_counts(const int32_t* __restrict__ counts, int q, int T) {
  if (q + 4 <= T) return *reinterpret_cast<const int4*>(counts + q);
  return make_int4(q < T ? counts[q] : 0, q + 1 < T ? counts[q + 1] : 0,
                   q + 2 < T ? counts[q + 2] : 0, 0);
}

__global__ __launch_bounds__(kScanThreads) void k_scan_sums(int T,
                                                            const int32_t* __restrict__ counts,
                                                            int4* __restrict__ part) {
  const int4 c = four_counts(counts, blockIdx.x * kScanChunk + 4 * (int)threadIdx.x, T);
  const ChunkTotals t = workgroup_totals(ChunkTotals{
      0, (long long)c.x + c.y + c.z + c.w, max(max(c.x, c.y), max(c.z, c.w))});
  if (threadIdx.x == 0)
    part[blockIdx.x] = make_int4((int)(t.total & 0xFFFFFFFFll), (int)(t.total >> 32), t.longest, 0);
}

__global__ __launch_bounds__(kScanThreads) void k_scan(int T, const int32_t* __restrict__ counts,
                                                       const int4* __restrict__ part,
                                                       int2* __restrict__ ranges, int capacity,
                                                       int32_t* __restrict__ status) {
  __shared__ long long s_wave[kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int base = blockIdx.x * kScanChunk;
  const int4 c = four_counts(counts, base + 4 * tid, T);
  ChunkTotals t{0, 0, 0};
  if (part) {
    for (int b = tid; b < (int)gridDim.x; b += kScanThreads) {
      const int4 p = part[b];
      const long long sum = (long long)(uint32_t)p.x | (long long)p.y << 32;
      t.total += sum;
      if (b < (int)blockIdx.x) t.before += sum;
      t.longest = max(t.longest, p.z);
    }
  } else {
    for (int q = 4 * tid; q < T; q += kScanChunk) {
      const int4 v = four_counts(counts, q, T);
      const long long sum = (long long)v.x + v.y + v.z + v.w;
      t.total += sum;
      if (q < base) t.before += sum;
      t.longest = max(t.longest, max(max(v.x, v.y), max(v.z, v.w)));
    }
  }
  t = workgroup_totals(t);
  const bool over = t.total > (long long)capacity;
  // the thread's place in its chunk
  const long long mine = (long long)c.x + c.y + c.z + c.w;
  long long incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const long long o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  long long begin = t.before + incl - mine;
  for (int w = 0; w < wave; ++w) begin += s_wave[w];
  // (ranges fit in int32 whenever they are written: P is then at most the int32 capacity)
  const int n[4] = {c.x, c.y, c.z, c.w};
  int b = (int)begin;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = base + 4 * tid + k;
    if (i < T) ranges[i] = over ? make_int2(0, 0) : make_int2(b, b + n[k]);
    b += n[k];
  }
  if (blockIdx.x == 0 && tid == 0) {
    status[0] = (int)min(t.total, (long long)INT32_MAX);
    status[1] = over ? 1 : 0;
    status[2] = t.longest;
    status[kNonfiniteOut] = status[kNonfinite];
  }
}

// Lane q of a kernel's group appends the kernel id to the buckets of the kernel's covered
// blocks q, q + 16, ... (row-major inside its block rectangle).  A lane's appends go out four at
// a time: each waits for its atomic's result only when all four are on their way.
__global__ __launch_bounds__(256) void k_scatter(Segs S, const int4* __restrict__ tile_rects,
                                                 const int2* __restrict__ ranges,
                                                 int32_t* __restrict__ cursors,
                                                 uint32_t* __restrict__ vals,
                                                 const int32_t* __restrict__ status) {
  constexpr int AHEAD = 4;
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int g = gid / kScatterLanes, q0 = gid % kScatterLanes;
  if (g >= S.K || status[1] != 0) return;
  const int j = binning_kernel(g, S.K);
  const int4 rc = tile_rects[j];
  const int n = rect_count(rc);
  if (q0 >= n) return;
  const SegGrid sg = seg_of_kernel(S, j);
  const int w = rc.z - rc.x + 1;
  for (int q = q0; q < n; q += AHEAD * kScatterLanes) {
    int pos[AHEAD];
    int2 rg[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      const int p = q + k * kScatterLanes;
      if (p < n) {
        const int t = sg.tile_offset + (rc.y + p / w) * sg.ntx + rc.x + p % w;
        pos[k] = atomicSub(&cursors[t], 1) - 1;  // the block's count runs down to zero
        rg[k] = ranges[t];
      }
    }
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
      if (q + k * kScatterLanes < n && pos[k] >= 0 && rg[k].x + pos[k] < rg[k].y)
        vals[rg[k].x + pos[k]] = (uint32_t)j;
  }
}

// The fit step's scatter into fixed-width buckets: entry t W + c of the pair storage, c the
// block's cursor, receives (kernel id << shift) | low, where low names the row the block's
// partial row of the kernel will be written to and read back from, so that no later pass has
// to search the sorted lists: low = q, the block's row-major index in the kernel's rectangle,
// for q < kSlots (row kSlots j + q), else kSlots + c (row kSlots K + t W + c).  A bucket that
// fills up sets the step's overflow flag (status word kStepFlags + parity of the step
// counter) and drops the entry -- the step then changes nothing.  The cursors start at zero
// (the fused render resets them).  The kernel's block rectangle comes from its model row
// (kernel_rects, the binning's own rule; a row with a NaN or infinite parameter covers no
// block) and is stored with its count for the step's Adam kernel, which gathers the
// kernel's partial rows over it.  The last workgroup copies the step counter into the status
// words and writes the step's Adam scalars, for the step's later kernels (three powf, which
// the first kernels' appends would wait for in their wave).
template <int LANES>
__global__ __launch_bounds__(256) void k_scatter_fixed(Segs S, const float* __restrict__ model,
                                                       int np, int4* __restrict__ tile_rects,
                                                       int32_t* __restrict__ counts,
                                                       int32_t* __restrict__ cursors,
                                                       uint32_t* __restrict__ vals, int width,
                                                       int shift, int32_t* __restrict__ status,
                                                       const int32_t* __restrict__ step,
                                                       smoe_adam_config adam,
                                                       float* __restrict__ scalars) {
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int t0 = step[0];
  if (blockIdx.x == gridDim.x - 1) {
    if (threadIdx.x == 0) {
      status[kStepShadow] = t0;
      adam_step_scalars(adam, t0, scalars);
    }
    return;
  }
  const int g = gid / LANES, q0 = gid % LANES;
  if (g >= S.K) return;  // (whole groups of LANES lanes: the shuffles stay inside one)
  const int j = binning_kernel(g, S.K);
  const SegGrid sg = seg_of_kernel(S, j);
  // every lane of the kernel's group reads the geometry; lane q0 also checks parameters
  // 5 + q0, 5 + q0 + LANES, ... for finiteness
  const float* p = model + (size_t)j * np;
  const float mux = p[0], muy = p[1], l11 = p[2], l21 = p[3], l22 = p[4];
  bool finite = __builtin_isfinite(mux) && __builtin_isfinite(muy) && __builtin_isfinite(l11) &&
                __builtin_isfinite(l21) && __builtin_isfinite(l22);
  for (int k = 5 + q0; k < np; k += LANES) finite = finite && __builtin_isfinite(p[k]);
  int bad = finite ? 0 : 1;
#pragma unroll
  for (int off = 1; off < LANES; off <<= 1) bad |= __shfl_xor(bad, off);
  int4 rc = make_int4(0, 0, -1, -1);
  if (!bad) rc = kernel_rects(mux, muy, l11, l21, l22, sg, S.r, S.box, S.trunc).tile;
  const int n = rect_count(rc);
  if (q0 == 0) {
    tile_rects[j] = rc;
    counts[j] = n;
  }
  if (n == 0) return;
  const int w = rc.z - rc.x + 1;
  for (int q = q0; q < n; q += LANES) {
    const int t = sg.tile_offset + (rc.y + q / w) * sg.ntx + rc.x + q % w;
    const int pos = atomicAdd(&cursors[t], 1);
    if (pos < width) {
      const uint32_t low = q < kSlots ? (uint32_t)q : (uint32_t)(kSlots + pos);
      vals[(size_t)t * width + pos] = ((uint32_t)j << shift) | low;
    } else {
      status[kStepFlags + (t0 & 1)] = 1;
    }
  }
}

// Orders every block's list by kernel id, writes the block-id keys and clears the block's
// counter.  A wave per block ranks a list of up to 64 ids in registers; a longer one is then
// taken by the workgroup's four waves together (sort_long).
constexpr int kSortBlocks = 4;
__global__ __launch_bounds__(64 * kSortBlocks) void k_sort_buckets(int T,
                                                                   const int2* __restrict__ ranges,
                                                                   uint32_t* __restrict__ vals,
                                                                   uint32_t* __restrict__ vals_alt,
                                                                   uint32_t* __restrict__ keys,
                                                                   int32_t* __restrict__ cursors) {
  __shared__ __align__(16) uint32_t s_rank[kSortBlocks][64];
  __shared__ LongSortScratch<kSortBlocks, 32768> s_long;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int t0 = blockIdx.x * kSortBlocks, t = t0 + wave;
  if (t < T) {
    const int2 rg = ranges[t];
    const int n = rg.y - rg.x;
    if (lane == 0) cursors[t] = 0;
    for (int i = lane; i < n; i += 64) keys[rg.x + i] = (uint32_t)t;
    if (n > 0 && n <= 64) rank_sort64(vals + rg.x, n, s_rank[wave]);
  }
  for (int k = 0; k < kSortBlocks && t0 + k < T; ++k) {
    const int2 rg = ranges[t0 + k];
    if (rg.y - rg.x > 64)
      sort_long(vals + rg.x, vals_alt + rg.x, rg.y - rg.x, 0, s_long);
  }
}

// A fit's first kernel: zero the bucket cursors and the status words (P, overflow, longest list,
// step shadow, the overflow flags and the non-finite flag), whatever the workspace held before.
__global__ void k_prepare_fit(int32_t* __restrict__ cursors, int n, int32_t* __restrict__ status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cursors[i] = 0;
  if (i < 8) status[i] = 0;
}

// The binning's first kernel: zero the per-block counters and the non-finite flag.
__global__ void k_fill_counts(int32_t* __restrict__ counts, int n, int32_t* __restrict__ status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) counts[i] = 0;
  if (i == 0) status[kNonfinite] = 0;
}

__global__ void k_copy_i32(const int32_t* __restrict__ src, int32_t* __restrict__ dst, int n) {
  const int i = threadIdx.x;
  if (i < n) dst[i] = src[i];
}

inline int cdiv(long long a, int b) { return (int)((a + b - 1) / b); }

void preprocess(int C, int order, const float* params, const Segs& S, const smoe_bins& b,
                int32_t* tile_counts, hipStream_t s) {
  with_lanes(S, [&](auto lanes) {
    constexpr int L = decltype(lanes)::value;
    k_preprocess<L><<<cdiv((long long)S.K * L, 256), 256, 0, s>>>(
        C, order, params, S, reinterpret_cast<int4*>(b.tile_rects),
        reinterpret_cast<int4*>(b.native_rects), b.counts, b.records, b.record_stride, tile_counts,
        b.status);
  });
}

}  // namespace

hipError_t launch_count(int C, int order, const float* params, const Segs& S,
                        const smoe_bins& b, hipStream_t s) {
  // Counters and the non-finite flag start from zero (a fill kernel rather than a memset
  // node, so that the step can be captured into a graph).
  k_fill_counts<<<cdiv(S.T, 256), 256, 0, s>>>(b.tile_counts, S.T, b.status);
  if (S.K > 0) {
    preprocess(C, order, params, S, b, b.tile_counts, s);
  }
  return hipGetLastError();
}

hipError_t launch_scan(const Segs& S, const smoe_bins& b, hipStream_t s) {
  const int chunks = cdiv(S.T, kScanChunk);
  // the chunks' sums go where the binning writes its keys last (if that holds them)
  int4* part = nullptr;
  if (S.T > kScanDirect && b.capacity / 4 >= chunks) {
    part = reinterpret_cast<int4*>(b.keys);
    k_scan_sums<<<chunks, kScanThreads, 0, s>>>(S.T, b.tile_counts, part);
  }
  k_scan<<<chunks, kScanThreads, 0, s>>>(S.T, b.tile_counts, part,
                                         reinterpret_cast<int2*>(b.ranges), b.capacity, b.status);
  return hipGetLastError();
}

hipError_t launch_prepare_fit(int C, int order, const float* params, const Segs& S,
                              const smoe_bins& b, hipStream_t s) {
  k_prepare_fit<<<cdiv(S.T, 256), 256, 0, s>>>(b.tile_counts, S.T, b.status);
  if (S.K > 0) {
    preprocess(C, order, params, S, b, nullptr, s);
  }
  return hipGetLastError();
}

hipError_t launch_scatter_fixed(const Segs& S, const smoe_bins& b, const float* model, int np,
                                int width, int shift, const int32_t* step,
                                const smoe_adam_config& adam, float* scalars, hipStream_t s) {
  with_lanes(S, [&](auto lanes) {
    constexpr int L = decltype(lanes)::value;
    k_scatter_fixed<L><<<cdiv((long long)S.K * L, 256) + 1, 256, 0, s>>>(
        S, model, np, reinterpret_cast<int4*>(b.tile_rects), b.counts, b.tile_counts, b.vals,
        width, shift, b.status, step, adam, scalars);
  });
  return hipGetLastError();
}

hipError_t launch_scatter(const Segs& S, const smoe_bins& b, hipStream_t s) {
  if (S.K > 0) {
    k_scatter<<<cdiv((long long)S.K * kScatterLanes, 256), 256, 0, s>>>(
        S, reinterpret_cast<const int4*>(b.tile_rects), reinterpret_cast<const int2*>(b.ranges),
        b.tile_counts, b.vals, b.status);
  }
  return hipGetLastError();
}

hipError_t launch_copy_status(const smoe_bins& b, int32_t* out4, hipStream_t s) {
  k_copy_i32<<<1, 64, 0, s>>>(b.status, out4, 4);
  return hipGetLastError();
}

hipError_t launch_bin(int C, int order, const float* params, const Segs& S, const smoe_bins& b,
                      hipStream_t s) {
  hipError_t e = launch_count(C, order, params, S, b, s);
  if (e == hipSuccess) e = launch_scan(S, b, s);
  if (e == hipSuccess) e = launch_scatter(S, b, s);
  if (e != hipSuccess) return e;
  k_sort_buckets<<<cdiv(S.T, kSortBlocks), 64 * kSortBlocks, 0, s>>>(
      S.T, reinterpret_cast<const int2*>(b.ranges), b.vals, b.vals_alt, b.keys, b.tile_counts);
  return hipGetLastError();
}

}  // namespace smoe
