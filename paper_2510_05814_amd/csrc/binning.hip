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
// A small single raster has the same arrays from its blocks' side instead, in one or two launches
// (k_block_lists).
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
// follows the same rule; its four lanes share out only what is short.
constexpr int kManyKernels = 16384;
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

// A kernel row's factor as its raster sees it (native sharpening: L / f, a correctly rounded
// binary32 division), whether every parameter is finite, and the blocks it covers (none if not:
// such a row takes part nowhere).
// The np parameters are loaded together: a loop that stops at the first bad one waits for each
// (k_block_lists at 16 blocks 8.1 -> 7.0 us, the render of 65536 kernels at 2048^2 79 -> 76.5).
constexpr int kRowMax = num_params(3, 1);
struct RowBoxes {
  float l11, l21, l22;
  bool finite;
  KernelRects rects;
};
__device__ __forceinline__ RowBoxes row_boxes(const float* __restrict__ p, int np,
                                              const SegGrid& sg, const Segs& S) {
  float v[kRowMax];
#pragma unroll
  for (int k = 0; k < kRowMax; ++k) v[k] = p[min(k, np - 1)];
  RowBoxes r;
  r.l11 = v[2];
  r.l21 = v[3];
  r.l22 = v[4];
  if (sg.sharpen != 1.0f) {
    r.l11 = r.l11 / sg.sharpen;
    r.l21 = r.l21 / sg.sharpen;
    r.l22 = r.l22 / sg.sharpen;
  }
  int bad = (__builtin_isfinite(r.l11) ? 0 : 1) | (__builtin_isfinite(r.l21) ? 0 : 1) |
            (__builtin_isfinite(r.l22) ? 0 : 1);
#pragma unroll
  for (int k = 0; k < kRowMax; ++k) bad |= __builtin_isfinite(v[k]) ? 0 : 1;
  r.finite = bad == 0;
  if (r.finite) {
    r.rects = kernel_rects(v[0], v[1], r.l11, r.l21, r.l22, sg, S.r, S.box, S.trunc);
  } else {
    r.rects.tile = r.rects.native = make_int4(0, 0, -1, -1);
  }
  return r;
}

// Where a non-finite row is reported: at once, in the status word (COUNT and BOXES), or, where
// no launch before this one has cleared the word, by the row's rectangle in tile_rects
// (MARK: kMarkedRow in .w; as empty as any, and k_block_lists replaces it).  MARK also clears
// the longest list, which k_block_lists raises.
constexpr int kMarkedRow = -2;
enum class Rows { COUNT, BOXES, MARK };

// SHARED: rasters with scales above 1, where the scale^2 output blocks of a native block have the
// same list.  The counters' atomics and the appends then go by native block -- its first output
// block stands for it -- and the other blocks take its count and rank its entries.  By output block
// against by native block: 16384 kernels on 4096^2 at scale 4 72.5 / 53.7 us, at scale 3 52.6 /
// 41.9, at scale 2 31.4 / 30.6; 700^2 at scale 8 120 / 67; in a batch of requests at scales 1 to 4
// (220 000 blocks) k_preprocess 84 / 34 and k_scatter 68 / 29 us.
inline bool shared_lists(const Segs& S) { return S.max_scale > 1; }

// Global id of the block counted for covered block (x, y): of the raster's blocks, or (SHARED) of
// the native ones.
template <bool SHARED>
__device__ __forceinline__ int covered_block(const SegGrid& sg, int x, int y) {
  if (SHARED) {
    x = native_first(x, sg.scale, sg.bx0);
    y = native_first(y, sg.scale, sg.by0);
  }
  return sg.tile_offset + y * sg.ntx + x;
}

// Every lane of a kernel's group reads the row and computes the output-block and native-block
// rectangles; lane 0 writes them and the count, lane q the q-th float4 of the render record,
// and (COUNT) lane q adds one to the counts of the kernel's covered blocks q, q +
// LANES, ... (row-major).  A row with a NaN or infinite parameter covers no block (it takes
// part nowhere) and sets the non-finite status word.
template <int LANES, Rows ROWS, bool SHARED>
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
  if (ROWS == Rows::MARK && gid == 0) status[2] = 0;
  if (g >= S.K) return;
  const int j = binning_kernel(g, S.K);
  const SegGrid sg = seg_of_kernel(S, j);
  const int ne = expert_floats(C, order);
  const float* p = params + (size_t)(sg.param_offset + (j - sg.kernel_offset)) * (6 + ne);
  const RowBoxes row = row_boxes(p, 6 + ne, sg, S);
  const int4 rc = row.rects.tile;
  if (lq == 0) {
    tile_rects[j] = ROWS == Rows::MARK && !row.finite ? make_int4(0, 0, -1, kMarkedRow) : rc;
    native_rects[j] = row.rects.native;
    counts[j] = rect_count(rc);
    if (ROWS != Rows::MARK && !row.finite) status[kNonfinite] = 1;
  }
  if (lq < rs / 4)
    write_record_quad(records + (size_t)j * rs, p, ne, lq, row.l11, row.l21, row.l22);
  if (ROWS == Rows::COUNT) {
    const int4 over = SHARED ? row.rects.native : rc;
    const int n = rect_count(over), w = over.z - over.x + 1;
    for (int q = lq; q < n; q += LANES)
      atomicAdd(&tile_counts[covered_block<SHARED>(sg, over.x + q % w, over.y + q / w)], 1);
  }
}

// Exclusive scan of the per-block counts into [begin, end) ranges, with P, the overflow flag
// and the longest list into status.  A chunk is kScanChunk consecutive blocks, four counts a
// thread; a workgroup takes one chunk, or `per` of them in turn; none waits for another.  What lies
// before its chunks, and the total (on an overflow every range is written empty), each workgroup
// sums for itself: from all the counts (part null), or from the chunks' sums that k_scan_sums
// left in part.  With a workgroup to a chunk, summing all the counts is quadratic in their number,
// so it serves up to kScanDirect blocks (4096^2 pixels: 256 KB read by each of 16 workgroups),
// where it saves a launch; beyond, where the storage has no room for the chunks' sums, by
// kScanDirect / kScanChunk workgroups (binning of 65536^2 with room for 4096 pairs: 25.4 ms by a
// workgroup a chunk, 11.1 by a single one for all, 3.4 by sixteen).
// One workgroup that walked all chunks took 7.7 us at 16384 blocks and 107 us for the 220 000 of a
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
                                                       const int4* __restrict__ part, int per,
                                                       int2* __restrict__ ranges, int capacity,
                                                       int32_t* __restrict__ status) {
  __shared__ long long s_wave[2][kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long first = (long long)blockIdx.x * per * kScanChunk;  // (the last may pass T)
  ChunkTotals t{0, 0, 0};
  if (part) {  // (one chunk a workgroup)
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
      if (q < first) t.before += sum;
      t.longest = max(t.longest, max(max(v.x, v.y), max(v.z, v.w)));
    }
  }
  t = workgroup_totals(t);
  const bool over = t.total > (long long)capacity;
  for (int k = 0; k < per && first + (long long)k * kScanChunk < T; ++k) {
    const int base = (int)(first + (long long)k * kScanChunk);
    const int4 c = four_counts(counts, base + 4 * tid, T);
    // the thread's place in its chunk
    const long long mine = (long long)c.x + c.y + c.z + c.w;
    long long incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const long long o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    if (lane == 63) s_wave[k & 1][wave] = incl;
    __syncthreads();  // (the one barrier a chunk: the next writes the other half)
    long long begin = t.before + incl - mine;
    for (int w = 0; w < kScanThreads / 64; ++w) {
      const long long n = s_wave[k & 1][w];
      if (w < wave) begin += n;
      t.before += n;
    }
    // (ranges fit in int32 whenever they are written: P is then at most the int32 capacity)
    const int n[4] = {c.x, c.y, c.z, c.w};
    int b = (int)begin;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = base + 4 * tid + i;
      if (at < T) ranges[at] = over ? make_int2(0, 0) : make_int2(b, b + n[i]);
      b += n[i];
    }
  }
  if (blockIdx.x == 0 && tid == 0) {
    status[0] = (int)min(t.total, (long long)INT32_MAX);
    status[1] = over ? 1 : 0;
    status[2] = t.longest;
    status[kNonfiniteOut] = status[kNonfinite];
  }
}

// Lane q of a kernel's LANES lanes appends the kernel id to the buckets of the kernel's covered
// blocks q, q + LANES, ... (row-major inside its block rectangle; rects: tile_rects, or (SHARED)
// native_rects).  A lane's appends go out four at
// a time: each waits for its atomic's result only when all four are on their way.
// Four lanes: of a row's first sixteen blocks; the sixteen lanes of four rows take the
// further blocks of each row together.  Measured, the whole binning with sixteen lanes a row / with
// four to the end of the row / with this: 65536 ordered rows of 6.6 blocks on 1024^2 87 / 60 / 59 us
// (in random order 65.5 / 70 / 70), 262144 on 2048^2 201 / 134 / 133, 20000 rows of 69 blocks 100 /
// 130 / 107; 4096 rows of 5.6 blocks 18.1 / 19.0 and 4000 of 117 blocks 72 / 178: with_lanes gives
// them sixteen.
template <int LANES, bool SHARED>
__global__ __launch_bounds__(256) void k_scatter(Segs S, const int4* __restrict__ rects,
                                                 const int2* __restrict__ ranges,
                                                 int32_t* __restrict__ cursors,
                                                 uint32_t* __restrict__ vals,
                                                 const int32_t* __restrict__ status) {
  constexpr int AHEAD = 4;
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int g = gid / LANES, q0 = gid % LANES;
  if (status[1] != 0) return;
  // the row's blocks q, q + stride, ... below n, AHEAD of them
  auto append = [&](const SegGrid& sg, int j, int4 rc, int n, int q, int stride) {
    const int w = rc.z - rc.x + 1;
    int pos[AHEAD];
    int2 rg[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      const int p = q + k * stride;
      if (p < n) {
        const int t = covered_block<SHARED>(sg, rc.x + p % w, rc.y + p / w);
        pos[k] = atomicSub(&cursors[t], 1) - 1;  // the block's count runs down to zero
        rg[k] = ranges[t];
      }
    }
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
      if (q + k * stride < n && pos[k] >= 0 && rg[k].x + pos[k] < rg[k].y)
        vals[rg[k].x + pos[k]] = (uint32_t)j;
  };
  int4 rc = make_int4(0, 0, -1, -1);
  int j = 0;
  if (g < S.K) {
    j = binning_kernel(g, S.K);
    rc = rects[j];
  }
  const int n = rect_count(rc);
  constexpr int FIRST = LANES * AHEAD;
  if (q0 < n) {
    const SegGrid sg = seg_of_kernel(S, j);
    for (int q = q0; q < (LANES == 16 ? n : min(n, FIRST)); q += FIRST)
      append(sg, j, rc, n, q, LANES);
  }
  if (LANES == 16) return;
  // (the lanes of a group of sixteen stay together here: n of a row is the same for them)
  static_assert(LANES == 16 || FIRST == 16, "the rest begins with block 16");
#pragma unroll 1
  for (int r = 0; r < 16 / LANES; ++r) {
    const int from = r * LANES, nr = __shfl(n, from, 16);
    if (nr <= FIRST) continue;
    const int jr = __shfl(j, from, 16);
    const int4 rr = make_int4(__shfl(rc.x, from, 16), __shfl(rc.y, from, 16),
                              __shfl(rc.z, from, 16), __shfl(rc.w, from, 16));
    const SegGrid sg = seg_of_kernel(S, jr);
    for (int q = FIRST + (threadIdx.x & 15); q < nr; q += 16 * AHEAD) append(sg, jr, rr, nr, q, 16);
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

// The block counted for block t (SHARED): the first of its native block.
__device__ __forceinline__ int counted_block(const Segs& S, int t) {
  const SegGrid sg = seg_of_tile(S, t);
  const int tx = (t - sg.tile_offset) % sg.ntx, ty = (t - sg.tile_offset) / sg.ntx;
  return covered_block<true>(sg, native_of(sg.bx0 + tx, sg.scale),
                             native_of(sg.by0 + ty, sg.scale));
}

// SHARED: the first block of each native block has been counted; its other blocks take its count.
__global__ __launch_bounds__(256) void k_spread_counts(Segs S, int32_t* __restrict__ tile_counts) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= S.T) return;
  const int first = counted_block(S, t);
  if (first != t) tile_counts[t] = tile_counts[first];
}

// Orders every block's list by kernel id, writes the block-id keys and clears the block's
// counter.  A wave per block ranks a list of up to kRankList ids; a longer one is then
// taken by the workgroup's four waves together (sort_long).  SHARED: the entries stand, in any
// order, in vals_alt at the place of the native block's first block, which nothing here
// writes; each block ranks them into its own place (its keys' place is the scratch then).
constexpr int kSortBlocks = 4;
template <bool SHARED>
__global__ __launch_bounds__(64 * kSortBlocks) void k_sort_buckets(Segs S,
                                                                   const int2* __restrict__ ranges,
                                                                   uint32_t* __restrict__ vals,
                                                                   uint32_t* __restrict__ vals_alt,
                                                                   uint32_t* __restrict__ keys,
                                                                   int32_t* __restrict__ cursors) {
  __shared__ __align__(16) LongSortScratch<kSortBlocks, 32768, 2048> s_long;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int t0 = blockIdx.x * kSortBlocks, t = t0 + wave, T = S.T;
  // the workgroup's ranges, one to a lane: a load in front of each list's turn below would be
  // most of what a short list costs (220 000 blocks 120 us against 89)
  const int2 mine = lane < kSortBlocks && t0 + lane < T ? ranges[t0 + lane] : make_int2(0, 0);
  auto range = [&](int k) {
    return make_int2(__builtin_amdgcn_readlane(mine.x, k), __builtin_amdgcn_readlane(mine.y, k));
  };
  if (t < T) {
    const int2 rg = range(wave);
    const int n = rg.y - rg.x;
    if (lane == 0) cursors[t] = 0;
    // (a quarter of s_long a wave: sort_long writes there only after a barrier of all four)
    uint32_t* s_rank = s_long.run + wave * kRankList;
    if (n > 0 && n <= kRankList) {
      const uint32_t* from = SHARED ? vals_alt + ranges[counted_block(S, t)].x : vals + rg.x;
      if (n <= 64) {
        const uint32_t e = lane < n ? from[lane] : 0xFFFFFFFFu;
        const int rank = rank64(e, n, s_rank);
        if (lane < n) {
          vals[rg.x + rank] = e;
          keys[rg.x + lane] = (uint32_t)t;
        }
      } else {
        rank_list<64>(from, vals + rg.x, n, s_rank, lane, wave_sync);
        for (int i = lane; i < n; i += 64) keys[rg.x + i] = (uint32_t)t;
      }
    } else if (!SHARED) {
      for (int i = lane; i < n; i += 64) keys[rg.x + i] = (uint32_t)t;
    }
  }
  for (uint64_t left = __ballot(mine.y - mine.x > kRankList); left != 0; left &= left - 1) {
    const int k = __builtin_ctzll(left);
    const int2 rg = range(k);
    const int n = rg.y - rg.x;
    if (!SHARED) {
      sort_long(vals + rg.x, vals_alt + rg.x, n, 0, s_long);
    } else {
      const uint32_t* from = vals_alt + ranges[counted_block(S, t0 + k)].x;
      for (int i = threadIdx.x; i < n; i += 64 * kSortBlocks) vals[rg.x + i] = from[i];
      __threadfence_block();
      __syncthreads();
      sort_long(vals + rg.x, keys + rg.x, n, 0, s_long);
      for (int i = threadIdx.x; i < n; i += 64 * kSortBlocks) keys[rg.x + i] = (uint32_t)(t0 + k);
    }
  }
}

// The whole ordering of a small raster in one kernel, by its blocks instead of its pairs: a
// block's list is read off the kernels' rectangles.  A lane holds a rectangle, and whether each
// of 64 kernels covers a block is one ballot, whose set bits are already in the order of the
// ids: no histogram, no atomics on counters, no sort.  Where a workgroup's lists begin it works
// out by itself, from the number of each rectangle's blocks that lie before its own.  The work
// grows with kernels times blocks (kListPairs), but a chunk of 64 kernels that misses the
// workgroup's blocks altogether -- neighbouring ids are neighbours in the image -- costs one
// test, and a kernel that covers every block costs what any other does, where the counters'
// atomics queue up.  What bounds it is the latency of its phases (loads, ballots, two
// scans, stores), so the rectangles of four chunks are loaded ahead (at 16384 kernels and 4096
// blocks 30.0 -> 24.4 us) -- and, where the kernels' order does not follow the image and every chunk
// has a few of every block's, the ballots and the chunks' turns at the end: ballots are gathered in
// lanes and stored together, and a lane then writes its own chunk's few entries (16384 kernels in
// random order on 1024x512 40.1 -> 26.6 us, in the image's order 22.3 -> 21.6; 4000 wide ones on
// 512^2 18 -> 16).  The figures against the other binning are with the rule below.
//
// ROWS_TOO: a single workgroup takes all blocks, and each lane works its kernel's row out itself
// (k_preprocess's work: one launch less).  Otherwise k_preprocess<MARK> has run, and a
// workgroup takes kListBlocks blocks, one for each of its waves.
struct ListArgs {
  Segs S;  // a single raster (no table)
  int C, order;
  const float* __restrict__ params;
  int4* __restrict__ tile_rects;
  int4* __restrict__ native_rects;
  int32_t* __restrict__ counts;
  float* __restrict__ records;
  int rs;
  int32_t* __restrict__ tile_counts;
  int2* __restrict__ ranges;
  uint32_t* __restrict__ keys;
  uint32_t* __restrict__ vals;
  int capacity;
  int32_t* __restrict__ status;
};
constexpr int kListWaves = 8, kListThreads = 64 * kListWaves, kListBlocks = kListWaves;
constexpr int kListMasks = 2048;  // ballots a workgroup keeps (blocks x chunks of 64 kernels)

// Lane LANE of (lo, hi) takes m (wave-uniform).
template <int LANE>
__device__ __forceinline__ void write_lane(uint64_t m, uint32_t& lo, uint32_t& hi) {
  asm("v_writelane_b32 %0, %1, %2" : "+v"(lo) : "s"((uint32_t)m), "n"(LANE));
  asm("v_writelane_b32 %0, %1, %2" : "+v"(hi) : "s"((uint32_t)(m >> 32)), "n"(LANE));
}

template <bool ROWS_TOO>
__global__ __launch_bounds__(kListThreads) void k_block_lists(ListArgs a) {
  __shared__ uint64_t s_mask[kListMasks];  // [block][chunk]
  __shared__ int s_list[kListThreads];     // a block's entries, then where they begin
  __shared__ int s_before[kListWaves], s_total[kListWaves], s_odd[kListWaves];
  __shared__ int s_scan[kListWaves], s_longest[kListWaves];
  const SegGrid sg = seg_grid_of(a.S.one);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.S.K, chunks = (K + 63) >> 6;
  const int t0 = ROWS_TOO ? 0 : blockIdx.x * kListBlocks;
  const int nb = ROWS_TOO ? a.S.T : min(kListBlocks, a.S.T - t0);
  // the workgroup's blocks: from (tx0, ty0) on in row-major order; inside [xa, xb] x [ty0, ty1]
  const int tx0 = t0 % sg.ntx, ty0 = t0 / sg.ntx, ty1 = (t0 + nb - 1) / sg.ntx;
  const int xa = ty0 == ty1 ? tx0 : 0, xb = ty0 == ty1 ? (t0 + nb - 1) % sg.ntx : sg.ntx - 1;

  int before = 0, total = 0, odd = 0;  // (at most kListPairs)
  // one chunk's rectangles against the blocks
  auto chunk = [&](int c, int4 rc) {
    const int n = rect_count(rc), w = rc.z - rc.x + 1;
    total += n;
    if (n > 0) {
      before += w * min(max(ty0 - rc.y, 0), rc.w - rc.y + 1);
      if (rc.y <= ty0 && ty0 <= rc.w) before += min(max(tx0 - rc.x, 0), w);
    }
    if (__ballot(n > 0 && rc.y <= ty1 && rc.w >= ty0 && rc.x <= xb && rc.z >= xa) != 0) {
      // lane b keeps block b's ballot (there are at most 64), and one store takes them all
      int tx = tx0, ty = ty0;
      uint32_t lo = 0, hi = 0;
      uint64_t row = __ballot(rc.y <= ty && ty <= rc.w);
      auto next = [&]() {
        const uint64_t m = row & __ballot(rc.x <= tx && tx <= rc.z);
        if (++tx == sg.ntx) {
          tx = 0;
          ++ty;
          row = __ballot(rc.y <= ty && ty <= rc.w);
        }
        return m;
      };
      if (ROWS_TOO) {
        for (int b = 0; b < nb; ++b) {
          const uint64_t m = next();
          lo = lane == b ? (uint32_t)m : lo;
          hi = lane == b ? (uint32_t)(m >> 32) : hi;
        }
      } else {  // (blocks past nb are worked out and not stored)
        write_lane<0>(next(), lo, hi);
        write_lane<1>(next(), lo, hi);
        write_lane<2>(next(), lo, hi);
        write_lane<3>(next(), lo, hi);
        write_lane<4>(next(), lo, hi);
        write_lane<5>(next(), lo, hi);
        write_lane<6>(next(), lo, hi);
        write_lane<7>(next(), lo, hi);
        static_assert(kListBlocks == 8, "a lane each");
      }
      if (lane < nb) s_mask[lane * chunks + c] = (uint64_t)hi << 32 | lo;
    } else if (lane < nb) {
      s_mask[lane * chunks + c] = 0;
    }
  };
  const int4 none = make_int4(0, 0, -1, -1);
  if (ROWS_TOO) {
    for (int c = wave; c < chunks; c += kListWaves) {
      const int j = 64 * c + lane;
      int4 rc = none;
      if (j < K) {
        const int ne = expert_floats(a.C, a.order);
        const float* p = a.params + (size_t)(sg.param_offset + j) * (6 + ne);
        const RowBoxes row = row_boxes(p, 6 + ne, sg, a.S);
        rc = row.rects.tile;
        odd |= row.finite ? 0 : 1;
        a.tile_rects[j] = rc;
        a.native_rects[j] = row.rects.native;
        a.counts[j] = rect_count(rc);
        for (int q = 0; q < a.rs / 4; ++q)
          write_record_quad(a.records + (size_t)j * a.rs, p, ne, q, row.l11, row.l21, row.l22);
      }
      chunk(c, rc);
    }
  } else {
    constexpr int AHEAD = 4;  // chunks on their way
    for (int c0 = wave; c0 < chunks; c0 += AHEAD * kListWaves) {
      int4 rc[AHEAD];
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        const int j = 64 * (c0 + k * kListWaves) + lane;
        rc[k] = a.tile_rects[min(j, K - 1)];
        if (j >= K) rc[k] = none;
      }
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        const int c = c0 + k * kListWaves;
        if (c >= chunks) break;
        if (rc[k].w == kMarkedRow) {
          odd = 1;
          if (blockIdx.x == 0) a.tile_rects[64 * c + lane] = none;
        }
        chunk(c, rc[k]);
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    before += __shfl_xor(before, off);
    total += __shfl_xor(total, off);
    odd |= __shfl_xor(odd, off);
  }
  if (lane == 0) {
    s_before[wave] = before;
    s_total[wave] = total;
    s_odd[wave] = odd;
  }
  __syncthreads();
  before = total = odd = 0;
  for (int v = 0; v < kListWaves; ++v) {
    before += s_before[v];
    total += s_total[v];
    odd |= s_odd[v];
  }
  const bool over = total > a.capacity;

  // the blocks' entries: a few chunks each, counted by a thread, or many, by a wave
  if (ROWS_TOO) {
    int n = 0;
    if (tid < nb)
      for (int c = 0; c < chunks; ++c) n += __popcll(s_mask[tid * chunks + c]);
    s_list[tid] = n;
  } else if (wave < nb) {
    int n = 0;
    for (int c = lane; c < chunks; c += 64) n += __popcll(s_mask[wave * chunks + c]);
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
    if (lane == 0) s_list[wave] = n;
  }
  __syncthreads();
  const int n = tid < nb ? s_list[tid] : 0;
  int incl = n, longest = n;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
    longest = max(longest, __shfl_xor(longest, off));
  }
  if (lane == 63) {
    s_scan[wave] = incl;
    s_longest[wave] = longest;
  }
  __syncthreads();
  int begin = before + incl - n;
  for (int v = 0; v < kListWaves; ++v) {
    if (v < wave) begin += s_scan[v];
    longest = max(longest, s_longest[v]);
  }
  if (tid < nb) {
    s_list[tid] = begin;
    a.ranges[t0 + tid] = over ? make_int2(0, 0) : make_int2(begin, begin + n);
    a.tile_counts[t0 + tid] = 0;
  }
  if (tid == 0) {
    if (ROWS_TOO) a.status[2] = longest;
    else atomicMax(&a.status[2], longest);
    if (blockIdx.x == 0) {
      a.status[0] = total;
      a.status[1] = over ? 1 : 0;
      a.status[kNonfiniteOut] = a.status[kNonfinite] = odd;
    }
  }
  if (over) return;  // (the same for all threads of all workgroups)
  __syncthreads();
  for (int b = wave; b < nb; b += kListWaves) {
    int pos = __builtin_amdgcn_readfirstlane(s_list[b]);
    for (int c0 = 0; c0 < chunks; c0 += 64) {
      const uint64_t mine = c0 + lane < chunks ? s_mask[b * chunks + c0 + lane] : 0;
      uint64_t left = __ballot(mine != 0);
      // Many chunks with an entry or two each (kernels in no order): a lane writes its own chunk's.
      const int own = __popcll(mine);
      if (__ballot(own > 4) == 0 && __popcll(left) > 4) {
        int at = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int o = __shfl_up(at, off);
          if (lane >= off) at += o;
        }
        const int all = __builtin_amdgcn_readlane(at, 63);
        at += pos - own;
        for (uint64_t m = mine; m != 0; m &= m - 1, ++at) {
          a.vals[at] = (uint32_t)(64 * (c0 + lane) + __builtin_ctzll(m));
          a.keys[at] = (uint32_t)(t0 + b);
        }
        pos += all;
        continue;
      }
      for (; left != 0; left &= left - 1) {
        const int c = __builtin_ctzll(left);
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)mine, c);
        const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(mine >> 32), c);
        const uint64_t m = (uint64_t)hi << 32 | lo;
        if (m >> lane & 1) {
          const int at = pos + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
          a.vals[at] = (uint32_t)(64 * (c0 + c) + lane);
          a.keys[at] = (uint32_t)(t0 + b);
        }
        pos += __popcll(m);
      }
    }
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

inline int cdiv(long long a, int b) { return (int)((a + b - 1) / b); }

template <Rows ROWS, bool SHARED = false>
void preprocess(int C, int order, const float* params, const Segs& S, const smoe_bins& b,
                hipStream_t s) {
  with_lanes(S, [&](auto lanes) {
    constexpr int L = decltype(lanes)::value;
    k_preprocess<L, ROWS, SHARED><<<cdiv((long long)S.K * L, 256), 256, 0, s>>>(
        C, order, params, S, reinterpret_cast<int4*>(b.tile_rects),
        reinterpret_cast<int4*>(b.native_rects), b.counts, b.records, b.record_stride,
        b.tile_counts, b.status);
  });
}

// Rasters whose lists k_block_lists makes.  Measured, the binning by counters and sorts against
// this one, kernels in the image's order / in random order: 64 kernels on 64^2 15.5 / 7.1 us and 15.0
// / 7.1, 1024 on 256^2 16.4 / 9.0 and 18.4 / 9.7, 4096 on 512^2 18.0 / 11.6 and 19.9 / 13.0, 8192 on
// 724^2 (2^24 pairs) 19.2 / 15.9 and 20.8 / 21.8, 16384 on 1024x512 (2^25) 24.1 / 21.7 and 25.6 /
// 26.7 -- there the gain is the wide kernels': 16384 with 376 000 entries 76 / 24 and 63 / 38, 2048 on
// 256^2 with 146 000 100 / 13 and 95 / 13, 4000 on 512^2 with 390 000 87 / 16 and 89 / 19.  Of 4, 8 and
// 16 blocks to a workgroup eight are the best at 512^2 (12.7 / 11.7 / 13.1 us before the ballots were
// gathered in lanes); four are 0.4 us faster at 256^2 and 7.7 us slower at 1024^2.
constexpr int kListKernels = kListMasks / kListBlocks * 64, kListTiles = 4096;
constexpr long long kListPairs = 1ll << 25;
inline bool lists_by_block(const Segs& S) {
  return !S.tab && S.K > 0 && S.K <= kListKernels && S.T <= kListTiles &&
         (long long)S.K * S.T <= kListPairs;
}
// ... and by a single workgroup, with their rows (at most 64 blocks): 16 ballots (64^2) 7.0 us and one launch,
// 64 about the time of the two launches, 256 14.5 us against 8.5.
inline bool lists_at_once(const Segs& S) {
  return S.K <= kListThreads && S.T <= kListThreads && cdiv(S.K, 64) * S.T <= 64;
}

hipError_t launch_block_lists(int C, int order, const float* params, const Segs& S,
                              const smoe_bins& b, hipStream_t s) {
  const ListArgs a{S,
                   C,
                   order,
                   params,
                   reinterpret_cast<int4*>(b.tile_rects),
                   reinterpret_cast<int4*>(b.native_rects),
                   b.counts,
                   b.records,
                   b.record_stride,
                   b.tile_counts,
                   reinterpret_cast<int2*>(b.ranges),
                   b.keys,
                   b.vals,
                   b.capacity,
                   b.status};
  if (lists_at_once(S)) {
    k_block_lists<true><<<1, kListThreads, 0, s>>>(a);
  } else {
    preprocess<Rows::MARK>(C, order, params, S, b, s);
    k_block_lists<false><<<cdiv(S.T, kListBlocks), kListThreads, 0, s>>>(a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_count(int C, int order, const float* params, const Segs& S,
                        const smoe_bins& b, hipStream_t s) {
  // Counters and the non-finite flag start from zero (a fill kernel rather than a memset
  // node, so that the step can be captured into a graph).
  k_fill_counts<<<cdiv(S.T, 256), 256, 0, s>>>(b.tile_counts, S.T, b.status);
  if (S.K > 0) {
    if (shared_lists(S)) {
      preprocess<Rows::COUNT, true>(C, order, params, S, b, s);
      k_spread_counts<<<cdiv(S.T, 256), 256, 0, s>>>(S, b.tile_counts);
    } else {
      preprocess<Rows::COUNT>(C, order, params, S, b, s);
    }
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
  const int per = part ? 1 : cdiv(chunks, kScanDirect / kScanChunk);
  k_scan<<<cdiv(chunks, per), kScanThreads, 0, s>>>(S.T, b.tile_counts, part, per,
                                                    reinterpret_cast<int2*>(b.ranges), b.capacity,
                                                    b.status);
  return hipGetLastError();
}

hipError_t launch_prepare_fit(int C, int order, const float* params, const Segs& S,
                              const smoe_bins& b, hipStream_t s) {
  k_prepare_fit<<<cdiv(S.T, 256), 256, 0, s>>>(b.tile_counts, S.T, b.status);
  if (S.K > 0) {
    preprocess<Rows::BOXES>(C, order, params, S, b, s);
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
  if (S.K == 0) return hipSuccess;
  const int2* ranges = reinterpret_cast<const int2*>(b.ranges);
  with_lanes(S, [&](auto lanes) {
    constexpr int L = decltype(lanes)::value;
    const int groups = cdiv((long long)S.K * L, 256);
    if (shared_lists(S))
      k_scatter<L, true><<<groups, 256, 0, s>>>(S, reinterpret_cast<const int4*>(b.native_rects),
                                                ranges, b.tile_counts, b.vals_alt, b.status);
    else
      k_scatter<L, false><<<groups, 256, 0, s>>>(S, reinterpret_cast<const int4*>(b.tile_rects),
                                                 ranges, b.tile_counts, b.vals, b.status);
  });
  return hipGetLastError();
}

hipError_t launch_bin(int C, int order, const float* params, const Segs& S, const smoe_bins& b,
                      hipStream_t s) {
  if (lists_by_block(S)) return launch_block_lists(C, order, params, S, b, s);
  hipError_t e = launch_count(C, order, params, S, b, s);
  if (e == hipSuccess) e = launch_scan(S, b, s);
  if (e == hipSuccess) e = launch_scatter(S, b, s);
  if (e != hipSuccess) return e;
  const int2* ranges = reinterpret_cast<const int2*>(b.ranges);
  if (shared_lists(S))
    k_sort_buckets<true><<<cdiv(S.T, kSortBlocks), 64 * kSortBlocks, 0, s>>>(
        S, ranges, b.vals, b.vals_alt, b.keys, b.tile_counts);
  else
    k_sort_buckets<false><<<cdiv(S.T, kSortBlocks), 64 * kSortBlocks, 0, s>>>(
        S, ranges, b.vals, b.vals_alt, b.keys, b.tile_counts);
  return hipGetLastError();
}

}  // namespace smoe
