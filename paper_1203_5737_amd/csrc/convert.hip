// CSR -> ARG-CSR conversion on the GPU (Sec. 3 of the paper).
//
// Step 1 (grouping) is a sequential scan; it runs on the host (plan.cpp), or
// on the device (group.hip) when the caller has row_ptr on
// the device only.  The kernels here run steps 2-4, every group independently:
//   chunks_kernel   step 2: chunk size c_g = min{c >= 1 : sum_r max(1,ceil(L_r/c)) <= T}
//                   (row-grouped CSR: c_g = max(1, longest row)) and
//                   t_r = max(1, ceil(L_r/c_g)) chunks per row;
//                   step 3: inclusive per-group prefix sum of t_r -> threadsMapping
//   offsets_kernel  exclusive scan of c_g*T over the groups -> groupInfo.offset,
//                   and the sizes the host checks
//   schedule_kernel the launch schedule: ascending indices of groups whose
//                   chunk loop is long (compaction by an exclusive scan)
//   fill_kernel     step 4: every slot (j, k) of a group -- element j of chunk
//   fill_long_kernel k at offset + j*T + k -- is written exactly once: the
//                   matching CSR element if chunk k's row has one there,
//                   otherwise the artificial zero (0, -1); the CSR elements
//                   pass through LDS so that reads and writes are coalesced
//                   (fill_long_kernel takes the blocks of long rows, tile by
//                   tile, from a list schedule_kernel makes); every CSR element
//                   passes through one of the two, which also check its column
//                   index against [0, n_cols).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <mutex>
#include <new>
#include <vector>

#include "common.hpp"
#include "group.hpp"
#include "mailbox.hpp"
#include "plan.hpp"
#include "schedule.hpp"
#include "scratch.hpp"
#include "values.hpp"

namespace argcsr {
namespace {

constexpr int kWaves = 4;             // waves per workgroup, one group per wave
constexpr int kMaxBlockDim = 1024;    // conversion accepts 1 <= T <= 1024
constexpr int kChunkBlocks = 2048;    // workgroups of chunks_kernel: all the GPU holds at once
constexpr int kScanBlock = 256;
constexpr int kScanBlocks = 128;      // workgroups of the offset and heavy scans
constexpr int kScanShare = kChunkBlocks / kScanBlocks;   // shares of groups each takes
constexpr int kMinStage = 256;        // CSR elements one fill wave stages in LDS
constexpr int kMaxStage = 2048;
constexpr int kMaxFillWaves = 4;
constexpr size_t kMaxFillLds = size_t(64) << 10;
constexpr int kLongSteps = 16;        // steps per LDS tile in fill_long_kernel
constexpr int kLongGrid = 4096;       // one-wave workgroups of fill_long_kernel

// Device-side state of one conversion, all zero at its start but for
// `groups`, which step 1 on the device writes.
struct Status {
  GroupCount groups;                  // step 1's, when it runs on the device
  int32_t scans_done;                 // workgroups of offsets_kernel that have finished
  int32_t pad;
  unsigned long long heavy;           // heavy groups of those
  unsigned long long long_tiles;      // and tiles of long groups (see fill_kernel)
};
static_assert(offsetof(Status, scans_done) == sizeof(GroupCount),
              "step 1 clears what follows `groups`, and nothing of it");

// Words the kernels hand to the host (a pinned slot, or device memory).
constexpr int kBoxGroups = 0, kBoxSlots = 1, kBoxHeavy = 2, kBoxBadRowPtr = 3, kBoxBadColumn = 4,
              kBoxNnz = 5, kBoxLong = 6;
constexpr int kBoxWords = Mailbox::kWords;

__global__ __launch_bounds__(64) void clear_words_kernel(int32_t* __restrict__ p, int32_t n) {
  for (int32_t i = threadIdx.x; i < n; i += 64) p[i] = 0;
}

// A device plan's tables into the caller's buffers: group records as 4
// words, then the threads mapping.
__global__ __launch_bounds__(256) void adopt_plan_kernel(const int32_t* __restrict__ groups,
                                                         int64_t group_words,
                                                         const int32_t* __restrict__ tm,
                                                         int64_t n_rows,
                                                         int32_t* __restrict__ out_groups,
                                                         int32_t* __restrict__ out_tm) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
  for (int64_t i = t; i < group_words; i += stride) out_groups[i] = groups[i];
  for (int64_t i = t; i < n_rows; i += stride) out_tm[i] = tm[i];
}

// CSR elements a fill wave stages in LDS: the blocks of chunks up to twice
// the matrix's mean chunk size (at least 4 and at most 32 elements a chunk).
__host__ __device__ inline int32_t fill_stage(int32_t T, int64_t n_slots, int32_t n_groups) {
  const int64_t chunks = int64_t(n_groups) * T;
  const int64_t mean_chunk = (n_slots + chunks - 1) / chunks;
  int32_t stage = kMinStage;
  while (stage < kMaxStage && stage < 128 * mean_chunk) stage *= 2;
  return stage;
}

// Tiles of kLongSteps steps that a group leaves to fill_long_kernel: a group
// whose chunks are longer than stage/64 elements may have blocks whose CSR
// range does not fit the stage.
__host__ __device__ inline int32_t long_tiles(int32_t c, int32_t stage) {
  return int64_t(c) * 64 > stage ? (c - 1) / kLongSteps + 1 : 0;
}

// LDS of one fill wave: the group's rows (RowTables), then the staged columns
// and values (the byte count keeps the next wave's region 8-byte aligned)
template <typename S>
__host__ __device__ inline size_t fill_lds_bytes(int32_t T, int32_t stage) {
  const size_t b = sizeof(int32_t) * (3 * size_t(T) + size_t(stage)) + sizeof(S) * size_t(stage);
  return (b + 7) & ~size_t(7);
}

// The first group of share i of n equal shares.
__device__ __forceinline__ int32_t share_begin(int32_t n_groups, int32_t i, int32_t n) {
  return int32_t(int64_t(n_groups) * i / n);
}

// Lengths of a group's rows: row l in lane l % 64, sub-row l / 64.
template <int SUB>
__device__ __forceinline__ void row_lengths(const int32_t* __restrict__ rp, int32_t first,
                                            int32_t size, uint32_t (&L)[SUB]) {
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const int l = s * 64 + lane_id();
    L[s] = l < size ? uint32_t(rp[first + l + 1] - rp[first + l]) : 0u;
  }
}

// Steps 2 + 3 of one group by the calling wave; returns its chunk size.
template <int SUB>
__device__ __forceinline__ uint32_t group_chunks(const uint32_t (&L)[SUB], int32_t first,
                                                 int32_t size, int32_t T, bool row_grouped,
                                                 int32_t* __restrict__ tm) {
  const int lane = lane_id();
  uint32_t my_nnz = 0;
  int my_longest = 0;
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    my_nnz += L[s];
    my_longest = int(L[s]) > my_longest ? int(L[s]) : my_longest;
  }
  const uint32_t total = wave_sum(my_nnz);          // row_ptr is int32: no overflow
  const uint32_t longest = uint32_t(wave_max(my_longest));

  // chunks of the group's rows at chunk size c (at most nnz + 1024 < 2^32)
  auto chunks_needed = [&](uint32_t c) {
    uint32_t need = 0;
#pragma unroll
    for (int s = 0; s < SUB; ++s)
      if (s * 64 + lane < size) need += L[s] > c ? (L[s] - 1u) / c + 1u : 1u;
    return wave_sum(need);
  };
  // binary search on the non-increasing chunks_needed(c) between two bounds:
  // no c below total/T fits, and c = longest (one chunk per row) always does;
  // since max(1, ceil(L/c)) <= L/c + 1, every c >= total/(T - size) fits too.
  // Row-grouped CSR, and a group of T rows, take one chunk per row.
  uint32_t lo = uint32_t((uint64_t(total) + uint32_t(T) - 1) / uint32_t(T));
  lo = lo < 1u ? 1u : lo;
  uint32_t hi = longest < 1u ? 1u : longest;
  if (row_grouped || size >= T) {
    lo = hi;
  } else {
    const uint32_t fit = uint32_t((uint64_t(total) + uint32_t(T - size) - 1) / uint32_t(T - size));
    if (fit < hi) hi = fit < 1u ? 1u : fit;
  }
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if (chunks_needed(mid) <= uint32_t(T)) hi = mid;
    else lo = mid + 1;
  }
  int carry = 0;
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const int l = s * 64 + lane;
    const int t = l < size ? (L[s] > lo ? int((L[s] - 1u) / lo + 1u) : 1) : 0;
    const int incl = wave_inclusive_scan(t) + carry;
    if (l < size) tm[first + l] = incl;
    carry = __builtin_amdgcn_readlane(incl, 63);
  }
  return lo;
}

// Steps 2 + 3.  Workgroup i takes the i-th of kChunkBlocks equal shares of
// the groups, its waves every fourth group of the share, and leaves the
// share's slots in share_slots[i]: the scan of the offsets then needs no pass
// of its own over the groups.  SUB = sub-rows of 64 rows a group may have.
// The group count is *n_dev when given (step 1 on the device), else n_host.
// Bound by each group's chain -- record, row offsets, two wave reductions,
// the search (0 to ~4 rounds of one reduction), the scan -- so a wave has the
// next group's row offsets and the record after that on their way while it
// works.  On the power-law matrix of 10^6 rows (63 517 groups) a wave per
// group with reductions through LDS and the rows read again in every round
// of the search took 32 us, this takes 18 us; on the 27-point stencil of 10^6
// rows (7813 groups of T = 128 rows) 8.5 and 7.3 us.
template <int SUB>
__global__ __launch_bounds__(kWaves * 64) void chunks_kernel(
    const int32_t* __restrict__ rp, argcsr_group_info* __restrict__ groups, int32_t n_host,
    const GroupCount* __restrict__ n_dev, int32_t T, int32_t row_grouped,
    int32_t* __restrict__ tm, int64_t* __restrict__ share_slots) {
  __shared__ int64_t wave_slots[kWaves];
  const int32_t n_groups = n_dev ? n_dev->n_groups : n_host;
  const int wv = wave_uniform(int(threadIdx.x >> 6));
  const int32_t g1 = share_begin(n_groups, int32_t(blockIdx.x) + 1, kChunkBlocks);
  int32_t g = share_begin(n_groups, int32_t(blockIdx.x), kChunkBlocks) + wv;
  int64_t slots = 0;
  int2 rec{0, 0}, next{0, 0};                       // first row, size
  uint32_t L[SUB];
  auto record = [&](int32_t i) {
    return i < g1 ? int2{groups[i].first_row, groups[i].size} : int2{0, 0};
  };
  rec = record(g);
  next = record(g + kWaves);
  row_lengths<SUB>(rp, rec.x, rec.y, L);
  for (; g < g1; g += kWaves) {
    uint32_t Ln[SUB];
    row_lengths<SUB>(rp, next.x, next.y, Ln);
    const int2 after = record(g + 2 * kWaves);
    const uint32_t c = group_chunks<SUB>(L, rec.x, rec.y, T, row_grouped != 0, tm);
    if (lane_id() == 0) groups[g].chunk_size = int32_t(c);
    slots += int64_t(c) * T;
    rec = next;
    next = after;
#pragma unroll
    for (int s = 0; s < SUB; ++s) L[s] = Ln[s];
  }
  if (lane_id() == 0) wave_slots[wv] = slots;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) slots += wave_slots[w];
    share_slots[blockIdx.x] = slots;
  }
}

void launch_chunks(const int32_t* rp, argcsr_group_info* groups, int32_t n_groups,
                   const GroupCount* n_dev, int32_t T, int32_t format, int32_t* tm,
                   int64_t* share_slots, hipStream_t s) {
  const dim3 grid(kChunkBlocks), block(kWaves * 64);
  const int32_t rg = format == ARGCSR_FORMAT_RG ? 1 : 0;
  auto* kern = T <= 64    ? &chunks_kernel<1>
               : T <= 128 ? &chunks_kernel<2>
               : T <= 256 ? &chunks_kernel<4>
                          : &chunks_kernel<16>;
  kern<<<grid, block, 0, s>>>(rp, groups, n_groups, n_dev, T, rg, tm, share_slots);
}

// Workgroup-wide exclusive scan and sum.
__device__ int64_t block_exclusive_scan(int64_t v, int64_t* total) {
  __shared__ int64_t wave_tot[kScanBlock / 64];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  int64_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t t = __shfl_up(incl, d, 64);
    if (lane >= d) incl += t;
  }
  if (lane == 63) wave_tot[w] = incl;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int i = 0; i < kScanBlock / 64; ++i) {
    if (i < w) before += wave_tot[i];
    all += wave_tot[i];
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

// Sums of v[0 .. at) and of v[at .. n).
__device__ void split_sums(const int64_t* __restrict__ v, int32_t at, int32_t n, int64_t* before,
                           int64_t* rest) {
  int64_t b = 0, r = 0;
#pragma unroll 8
  for (int32_t i = threadIdx.x; i < n; i += kScanBlock) {
    const int64_t x = v[i];
    if (i < at) b += x;
    else r += x;
  }
  (void)block_exclusive_scan(b, before);
  (void)block_exclusive_scan(r, rest);
}

// Offsets (an exclusive scan of c_g*T over the groups), the heavy groups and
// the long tiles of every workgroup's part, and, by the workgroup that
// finishes last, the sizes for the host.  A workgroup takes kScanShare consecutive shares of
// chunks_kernel and sums the shares before them itself, so the scan is one
// launch.  Few workgroups: each adds to the counters of `st`, and atomics on
// one cache line take turns at about 12 ns each.
__global__ __launch_bounds__(kScanBlock) void offsets_kernel(
    argcsr_group_info* __restrict__ groups, int32_t n_host, const GroupCount* __restrict__ n_dev,
    int32_t T, const int64_t* __restrict__ share_slots, int64_t* __restrict__ heavy_parts,
    int64_t* __restrict__ long_parts, Status* __restrict__ st, const int32_t* __restrict__ rp,
    int32_t n_rows, int64_t* __restrict__ box) {
  const int32_t n_groups = n_dev ? n_dev->n_groups : n_host;
  const int32_t b = int32_t(blockIdx.x);
  int64_t off, rest;
  split_sums(share_slots, b * kScanShare, kChunkBlocks, &off, &rest);
  const int64_t slots = off + rest;
  const int32_t heavy_chunk = heavy_chunk_for(T, slots, n_groups);
  const int32_t g0 = share_begin(n_groups, b * kScanShare, kChunkBlocks);
  const int32_t g1 = share_begin(n_groups, (b + 1) * kScanShare, kChunkBlocks);
  const int32_t stage = fill_stage(T, slots > 0 ? slots : 1, n_groups > 0 ? n_groups : 1);
  int32_t heavy = 0;
  int64_t tiles = 0;
  for (int32_t i = g0; i < g1; i += kScanBlock) {
    const int32_t g = i + int32_t(threadIdx.x);
    const int32_t c = g < g1 ? groups[g].chunk_size : 0;
    int64_t all;
    const int64_t mine = off + block_exclusive_scan(int64_t(c) * T, &all);
    if (g < g1) groups[g].offset = int32_t(mine);    // the host checks the total
    heavy += c > heavy_chunk;
    tiles += long_tiles(c, stage);
    off += all;
  }
  int64_t part_heavy, part_tiles;
  (void)block_exclusive_scan(heavy, &part_heavy);
  (void)block_exclusive_scan(tiles, &part_tiles);
  if (threadIdx.x == 0) {
    heavy_parts[b] = part_heavy;
    long_parts[b] = part_tiles;
    if (part_heavy) atomicAdd(&st->heavy, (unsigned long long)part_heavy);
    if (part_tiles) atomicAdd(&st->long_tiles, (unsigned long long)part_tiles);
    __threadfence();
    if (atomicAdd(&st->scans_done, 1) == kScanBlocks - 1) {
      __threadfence();
      box[kBoxGroups] = n_groups;
      box[kBoxSlots] = slots;
      box[kBoxHeavy] = int64_t(atomicAdd(&st->heavy, 0ull));
      box[kBoxLong] = int64_t(atomicAdd(&st->long_tiles, 0ull));
      box[kBoxBadRowPtr] = n_dev ? n_dev->bad : 0;
      box[kBoxNnz] = n_dev ? rp[n_rows] : 0;
    }
  }
}

// The launch schedule and the fill's list of long tiles: every part of
// offsets_kernel writes the indices of its heavy groups (`heavy` may be NULL)
// and the (group, first step) of its long tiles, ascending, behind those of
// the parts before it.  7 us on the power-law matrix of 10^6 rows (29 000
// tiles).  When fill_kernel appended the tiles with one device atomic per
// group, those took turns on their cache line: it took 59 us there, without
// them 53.
constexpr int32_t kLaneTiles = 8;
__global__ __launch_bounds__(kScanBlock) void schedule_kernel(
    const argcsr_group_info* __restrict__ groups, int32_t n_groups, int32_t heavy_chunk,
    int32_t stage, const int64_t* __restrict__ heavy_parts,
    const int64_t* __restrict__ long_parts, int32_t* __restrict__ heavy,
    int2* __restrict__ long_list) {
  const int32_t b = int32_t(blockIdx.x);
  const bool any_heavy = heavy && heavy_parts[b] != 0, any_long = long_parts[b] != 0;
  if (!any_heavy && !any_long) return;
  int64_t at_heavy = 0, at_long = 0, rest;
  if (any_heavy) split_sums(heavy_parts, b, kScanBlocks, &at_heavy, &rest);
  if (any_long) split_sums(long_parts, b, kScanBlocks, &at_long, &rest);
  const int32_t g0 = share_begin(n_groups, b * kScanShare, kChunkBlocks);
  const int32_t g1 = share_begin(n_groups, (b + 1) * kScanShare, kChunkBlocks);
  for (int32_t i = g0; i < g1; i += kScanBlock) {
    const int32_t g = i + int32_t(threadIdx.x);
    const int32_t c = g < g1 ? groups[g].chunk_size : 0;
    int64_t all;
    if (any_heavy) {
      const int64_t at = at_heavy + block_exclusive_scan(c > heavy_chunk ? 1 : 0, &all);
      if (c > heavy_chunk) heavy[at] = g;
      at_heavy += all;
    }
    if (any_long) {
      const int32_t tiles = long_tiles(c, stage);
      const int64_t at = at_long + block_exclusive_scan(tiles, &all);
      // a lane writes a few entries itself, the wave those of a longer group
      if (tiles <= kLaneTiles)
        for (int32_t t = 0; t < tiles; ++t) long_list[at + t] = int2{g, t * kLongSteps};
      for (uint64_t big = __ballot(tiles > kLaneTiles); big; big &= big - 1) {
        const int from = __builtin_ctzll(big);
        const int32_t n = __builtin_amdgcn_readlane(tiles, from);
        const int32_t first = __builtin_amdgcn_readlane(int32_t(at), from);
        const int32_t group = __builtin_amdgcn_readlane(g, from);
        for (int32_t t = lane_id(); t < n; t += 64)
          long_list[first + t] = int2{group, t * kLongSteps};
      }
      at_long += all;
    }
  }
}

// The rows of a group in the wave's LDS: where each starts in the CSR arrays
// and its length, and per chunk a mark where a row's chunks begin.
struct RowTables {
  int32_t* start;     // [T]
  int32_t* len;       // [T]
  int32_t* mark;      // [T]: chunk << kRowBits | row at a row's first chunk, else 0
};
constexpr int kRowBits = 10;
static_assert(kMaxBlockDim <= 1 << kRowBits, "marks hold a chunk and a row");

__device__ __forceinline__ RowTables row_tables(int32_t* lds, int32_t T) {
  return RowTables{lds, lds + T, lds + 2 * T};
}

__device__ __forceinline__ void load_rows(const argcsr_group_info& gi,
                                          const int32_t* __restrict__ rp,
                                          const int32_t* __restrict__ tm, int32_t T, int lane,
                                          const RowTables& t) {
  for (int k = lane; k < T; k += 64) t.mark[k] = 0;
  wave_lds_sync();
  for (int l = lane; l < gi.size; l += 64) {
    const int32_t r = gi.first_row + l;
    const int32_t begin = l == 0 ? 0 : tm[r - 1];
    const int32_t first = rp[r];
    t.start[l] = first;
    t.len[l] = rp[r + 1] - first;
    t.mark[begin] = begin << kRowBits | l;
  }
  wave_lds_sync();
}

// Where the elements of chunk k of the group start in the CSR arrays and how
// many there are (0 for free chunks, k >= n_mapped).  The last mark at or
// before a chunk names its row and the row's first chunk: a running maximum
// over the chunks, `carry` taking it from one block of 64 to the next.  A loop
// over the chunks of each row, by the row's lane, runs as long as the group's
// row of most chunks, with one lane at work: fill_kernel took 53 us with it on
// the power-law matrix of 10^6 rows and fill_long_kernel 25, now 37 and 19.
struct ChunkSource {
  int32_t start, len;
};
__device__ __forceinline__ ChunkSource chunk_source(const RowTables& t, int32_t k, int32_t T,
                                                    int32_t n_mapped, int32_t c, int32_t* carry) {
  int32_t m = wave_inclusive_max(k < T ? t.mark[k] : 0);
  m = m > *carry ? m : *carry;
  *carry = __builtin_amdgcn_readlane(m, 63);
  const int32_t row = m & ((1 << kRowBits) - 1);
  if (k >= n_mapped) return ChunkSource{0, 0};
  const int32_t skip = (k - (m >> kRowBits)) * c;     // elements of the row's chunks before
  const int32_t left = t.len[row] - skip;
  return ChunkSource{t.start[row] + skip, left < 0 ? 0 : left < c ? left : c};
}

// The CSR range [lo, lo + extent) that holds the elements of the wave's 64
// chunks (start, len per lane); extent 0 when they have none.
__device__ inline int32_t block_extent(int32_t start, int32_t len, int32_t* lo_out) {
  const int32_t lo = INT32_MAX - wave_max(len > 0 ? INT32_MAX - start : 0);
  const int32_t hi = wave_max(len > 0 ? start + len : 0);
  *lo_out = lo;
  return hi > lo ? hi - lo : 0;
}

// Step 4, one wave per group.  The wave takes the group's chunks 64 at a
// time.  The elements of 64 consecutive chunks form one contiguous CSR range
// (a row's chunks follow each other, and so do the rows), so when that range
// fits the wave's stage of `stage` elements the wave copies it into LDS with coalesced loads,
// converting the values to their storage type, and then writes the block's
// slots step by step, 64 consecutive slots per store, each lane taking its
// chunk's element from LDS.  Blocks whose range is longer than the stage are
// left to fill_long_kernel.  Every staged column index is checked
// against [0, n_cols) (a negative one wraps above the limit as unsigned).
template <int DT>
__global__ __launch_bounds__(kMaxFillWaves * 64) void fill_kernel(
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
    const double* __restrict__ val, const argcsr_group_info* __restrict__ groups,
    int32_t n_groups, int32_t n_cols, int32_t T, const int32_t* __restrict__ tm, int32_t stage,
    int64_t* __restrict__ box, int32_t* __restrict__ columns,
    typename Val<DT>::storage* __restrict__ values) {
  using S = typename Val<DT>::storage;
  extern __shared__ int32_t fill_lds[];   // per wave: RowTables, stage
  const int lane = lane_id();
  const int w = wave_uniform(int(threadIdx.x >> 6));
  const size_t wave_bytes = fill_lds_bytes<S>(T, stage);
  int32_t* lds = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(fill_lds) + w * wave_bytes);
  const RowTables rows = row_tables(lds, T);
  int32_t* stage_col = lds + 3 * T;
  S* stage_val = reinterpret_cast<S*>(stage_col + stage);
  const int g = blockIdx.x * (blockDim.x >> 6) + w;
  if (g >= n_groups) return;
  const argcsr_group_info gi = groups[g];
  const int32_t c = gi.chunk_size;
  const int32_t n_mapped = tm[gi.first_row + gi.size - 1];
  load_rows(gi, rp, tm, T, lane, rows);
  const uint32_t limit = uint32_t(n_cols);
  bool bad = false;
  int32_t carry = 0;
  for (int32_t k0 = 0; k0 < T; k0 += 64) {
    const int32_t k = k0 + lane;
    const bool mine = k < T;
    const auto [start, len] = chunk_source(rows, k, T, n_mapped, c, &carry);
    int32_t lo;
    const int32_t extent = block_extent(start, len, &lo);
    const int64_t dst0 = int64_t(gi.offset) + k;
    if (extent <= stage) {
#pragma unroll 8
      for (int32_t p = lane; p < extent; p += 64) {
        const int32_t cp = col[lo + p];
        bad |= uint32_t(cp) >= limit;
        stage_col[p] = cp;
        stage_val[p] = Val<DT>::from_f64(val[lo + p]);
      }
      wave_lds_sync();
      const int32_t rel = start - lo;
      for (int32_t j = 0; j < c; ++j) {
        if (!mine) continue;
        const int64_t dst = dst0 + int64_t(j) * T;
        if (j < len) {
          columns[dst] = stage_col[rel + j];
          values[dst] = stage_val[rel + j];
        } else {
          columns[dst] = -1;
          values[dst] = S(0);
        }
      }
      wave_lds_sync();   // the next block overwrites the stage
    }
  }
  if (__ballot(bad) != 0 && lane == 0) box[kBoxBadColumn] = 1;
}

// Step 4 for the blocks fill_kernel leaves: those whose CSR range is longer
// than the stage, from the list of (group, first step) tiles that
// schedule_kernel made.  One-wave workgroups stride over the list; an item moves kLongSteps steps of the group's long
// blocks through LDS: each load instruction reads kLongSteps consecutive
// elements of each of 64/kLongSteps chunks (a lane past its chunk's end reads
// an element of the block and keeps the padding value, so the loads carry no
// branch and are issued together), and each store writes one step of the 64
// chunks, 64 consecutive slots.  The column indices of the elements it moves
// are checked as in fill_kernel.
template <int DT>
__global__ __launch_bounds__(64) void fill_long_kernel(
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
    const double* __restrict__ val, const argcsr_group_info* __restrict__ groups,
    int32_t n_cols, int32_t T, const int32_t* __restrict__ tm, int32_t stage,
    int64_t* __restrict__ box, const int2* __restrict__ long_list, int32_t n_items,
    int32_t* __restrict__ columns, typename Val<DT>::storage* __restrict__ values) {
  using S = typename Val<DT>::storage;
  constexpr int kPer = 64 / kLongSteps;           // chunks per load instruction
  __shared__ int32_t tile_col[kLongSteps][65];    // [step][chunk], padded rows
  __shared__ S tile_val[kLongSteps][65];
  __shared__ int32_t src_start[64], src_len[64];  // of the block's chunks
  extern __shared__ int32_t long_tables[];        // RowTables
  const RowTables rows = row_tables(long_tables, T);
  const int lane = lane_id();
  const int jj = lane % kLongSteps, kq = lane / kLongSteps;
  const uint32_t limit = uint32_t(n_cols);
  bool bad = false;
  for (int32_t i = blockIdx.x; i < n_items; i += gridDim.x) {
    const argcsr_group_info gi = groups[long_list[i].x];
    const int32_t j0 = long_list[i].y;
    const int32_t c = gi.chunk_size;
    const int32_t n_mapped = tm[gi.first_row + gi.size - 1];
    load_rows(gi, rp, tm, T, lane, rows);
    int32_t carry = 0;
    for (int32_t k0 = 0; k0 < T; k0 += 64) {
      const int32_t k = k0 + lane;
      const auto [start, len] = chunk_source(rows, k, T, n_mapped, c, &carry);
      int32_t lo;
      if (block_extent(start, len, &lo) <= stage) continue;
      src_start[lane] = start;
      src_len[lane] = len;
      wave_lds_sync();
      int32_t cv[kLongSteps];
      double v[kLongSteps];
      bool ok[kLongSteps];
#pragma unroll
      for (int it = 0; it < kLongSteps; ++it) {
        const int32_t kl = it * kPer + kq;          // a chunk at or past T has no elements
        const int32_t j = j0 + jj;
        ok[it] = j < src_len[kl];
        const int32_t e = ok[it] ? src_start[kl] + j : lo;
        cv[it] = col[e];
        v[it] = val[e];
        bad |= ok[it] && uint32_t(cv[it]) >= limit;
      }
#pragma unroll
      for (int it = 0; it < kLongSteps; ++it) {
        const int32_t kl = it * kPer + kq;          // chunk within the block
        tile_col[jj][kl] = ok[it] ? cv[it] : -1;
        tile_val[jj][kl] = ok[it] ? Val<DT>::from_f64(v[it]) : S(0);
      }
      wave_lds_sync();
      const int32_t steps = c - j0 < kLongSteps ? c - j0 : kLongSteps;
      if (k < T)
#pragma unroll 4
        for (int32_t u = 0; u < steps; ++u) {
          const int64_t dst = int64_t(gi.offset) + int64_t(j0 + u) * T + k;
          columns[dst] = tile_col[u][lane];
          values[dst] = tile_val[u][lane];
        }
      wave_lds_sync();   // the next block or item overwrites the tile and tables
    }
  }
  if (__ballot(bad) != 0 && lane == 0) box[kBoxBadColumn] = 1;
}

// Small stages leave room for 4 waves per workgroup, which the many short
// groups of irregular matrices need to hide their latency, as long as the
// waves' LDS stays within the 64 KB any launch may ask for (T = 1024: 2).
template <int DT>
void launch_fill(hipStream_t s, const int32_t* rp, const int32_t* col, const double* val,
                 int32_t stage, int64_t* box, const int2* long_list, int32_t n_long,
                 const argcsr_matrix* out) {
  using S = typename Val<DT>::storage;
  const int32_t T = out->block_dim;
  int waves = stage <= 512 ? kMaxFillWaves : 1;
  while (waves > 1 && fill_lds_bytes<S>(T, stage) * size_t(waves) > kMaxFillLds) waves /= 2;
  const size_t lds = fill_lds_bytes<S>(T, stage) * size_t(waves);
  const uint32_t blocks = uint32_t((int64_t(out->n_groups) + waves - 1) / waves);
  fill_kernel<DT><<<dim3(blocks), 64 * waves, lds, s>>>(
      rp, col, val, out->groups, out->n_groups, out->n_cols, T, out->threads_mapping, stage, box,
      out->columns, static_cast<S*>(out->values));
  if (n_long > 0)
    fill_long_kernel<DT><<<dim3(uint32_t(std::min(n_long, kLongGrid))), 64,
                           sizeof(int32_t) * 3 * size_t(T), s>>>(
        rp, col, val, out->groups, out->n_cols, T, out->threads_mapping, stage, box, long_list,
        n_long, out->columns, static_cast<S*>(out->values));
}

}  // namespace
}  // namespace argcsr

// A device plan (argcsr_plan_device_keep): steps 1-3 of one matrix kept on
// the device for argcsr_convert_planned, and the sizes of the result.
// Its buffers are one block of scratch, unused on the device whenever the plan
// is (planning and every conversion with it wait for their own work).
// The group table has room for one group a row, because the number of groups
// is only known to the device while the plan is made.
struct argcsr_device_plan {
  int32_t n_rows = 0, block_dim = 0, desired_chunk_size = 0, format = 0;
  int32_t n_groups = 0, n_heavy = 0;
  int64_t n_slots = 0, nnz = 0, n_long = 0;
  argcsr_group_info* groups = nullptr;    // complete, offsets included
  int32_t* tm = nullptr;                  // threads mapping
  int64_t* heavy_parts = nullptr;         // heavy groups per part of offsets_kernel,
                                          // then long tiles per part
  argcsr::DeviceScratch block;            // holds them
};

// Fixed scratch of argcsr_convert_noalloc: one copy per GPU (this process's
// code object), held until the process ends.  Host code reaches it only
// through the address hipGetSymbolAddress returns for the current device.
constexpr size_t kHeadBytes = 256;        // Status and the result words
constexpr size_t kNoAllocExtra = 32768;   // head, shares and parts
constexpr size_t kNoAllocScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocExtra + kNoAllocScratchBytes];

namespace argcsr {
namespace {

// Device scratch of one conversion: a head of kHeadBytes (Status and, for
// argcsr_convert_noalloc, the result words), the slots of the shares of
// chunks_kernel, the heavy groups and long tiles of the parts of
// offsets_kernel, and the fill's list of long tiles.  Entries of that
// list: a group makes them only when its chunk size c exceeds
// stage/64 >= kMinStage/64 = 4, and then ceil(c/16) <= c/4 of them, so all
// groups together make at most n_slots/(4T).
static_assert(kMinStage / 64 >= 4 && kLongSteps == 16, "long-list bound");
static_assert(sizeof(Status) + sizeof(int64_t) * kBoxWords <= kHeadBytes, "head of the scratch");
static_assert(kHeadBytes + sizeof(int64_t) * (kChunkBlocks + 2 * kScanBlocks) <= kNoAllocExtra,
              "head and shares of the fixed scratch");
constexpr size_t kShareBytes = sizeof(int64_t) * (kChunkBlocks + 2 * kScanBlocks);

int64_t long_capacity(int64_t n_slots, int32_t T) { return n_slots / (4 * int64_t(T)) + 1; }

size_t convert_scratch(int64_t n_slots, int32_t T) {
  return kHeadBytes + kShareBytes + 2 * sizeof(int32_t) * size_t(long_capacity(n_slots, T));
}

// The result words of one conversion: a pinned slot, or (fixed) words of the
// device scratch that are copied back.
struct ResultBox {
  Mailbox mail;
  int64_t* dev = nullptr;
  int64_t word[kBoxWords] = {};
  bool fixed = false;
  int init(int64_t* fixed_words, hipStream_t s) {
    fixed = fixed_words != nullptr;
    if (fixed) {
      dev = fixed_words;
      return ARGCSR_OK;
    }
    const int rc = mail.init(s);
    dev = mail.device();
    return rc;
  }
  // waits for the stream and reads the words (kernels queued later may write
  // them again; idle() after the last read)
  int read(hipStream_t s) {
    hipError_t e = hipSuccess;
    if (fixed) e = hipMemcpyAsync(word, dev, sizeof(word), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ARGCSR_EHIP, "conversion: %s", hipGetErrorString(e));
    if (!fixed)
      for (int i = 0; i < kBoxWords; ++i) word[i] = mail.word(i);
    return ARGCSR_OK;
  }
  void idle() { mail.idle(); }
};

// Steps 1-3 of n_rows > 0 rows on the device, and the sizes of the result
// (one wait for the stream).  A host copy of the row offsets, when given, is
// checked while the device works: 10^6 rows take the host 37 us, the device 45
// or more.
int build_plan(int32_t n_rows, const int32_t* row_ptr, int32_t T, int32_t desired, int32_t format,
               int32_t region_rows, const int32_t* regions, hipStream_t s, argcsr_device_plan* p,
               const int32_t* row_ptr_host = nullptr) {
  const size_t groups_b = sizeof(argcsr_group_info) * size_t(n_rows);
  const size_t tm_b = (sizeof(int32_t) * size_t(n_rows) + 15) / 16 * 16;
  ResultBox box;
  int rc = box.init(nullptr, s);
  if (rc) return rc;
  DeviceScratch work;
  rc = p->block.alloc(groups_b + tm_b + kShareBytes + sizeof(Status), s);
  if (rc == ARGCSR_OK)
    rc = work.alloc(group_work_bytes(n_rows, T, format, region_rows, regions), s);
  if (rc) return rc;
  char* base = static_cast<char*>(p->block.ptr());
  p->groups = reinterpret_cast<argcsr_group_info*>(base);
  p->tm = reinterpret_cast<int32_t*>(base + groups_b);
  auto* share_slots = reinterpret_cast<int64_t*>(base + groups_b + tm_b);
  p->heavy_parts = share_slots + kChunkBlocks;
  auto* st = reinterpret_cast<Status*>(p->heavy_parts + 2 * kScanBlocks);
  rc = group_on_device(n_rows, row_ptr, T, desired, format, region_rows, regions, p->groups,
                       &st->groups, &st->scans_done,
                       int64_t((sizeof(Status) - offsetof(Status, scans_done)) / sizeof(int32_t)),
                       work.ptr(), s);
  if (rc) return rc;
  launch_chunks(row_ptr, p->groups, 0, &st->groups, T, format, p->tm, share_slots, s);
  offsets_kernel<<<kScanBlocks, kScanBlock, 0, s>>>(p->groups, 0, &st->groups, T, share_slots,
                                                    p->heavy_parts, p->heavy_parts + kScanBlocks, st,
                                                    row_ptr, n_rows, box.dev);
  ARGCSR_HIP(hipGetLastError());
  const int host_rc = row_ptr_host ? check_row_ptr(n_rows, row_ptr_host) : ARGCSR_OK;
  rc = box.read(s);
  if (rc) return rc;
  p->block.idle();
  work.idle();
  box.idle();
  if (host_rc) return host_rc;
  if (box.word[kBoxBadRowPtr])
    return fail(ARGCSR_EINVAL, "row_ptr does not start at 0 or decreases");
  if (row_ptr_host && int64_t(row_ptr_host[n_rows]) != box.word[kBoxNnz])
    return fail(ARGCSR_EINVAL, "row_ptr_host ends at %d, row_ptr at %lld", row_ptr_host[n_rows],
                (long long)box.word[kBoxNnz]);
  p->n_rows = n_rows;
  p->block_dim = T;
  p->desired_chunk_size = format == ARGCSR_FORMAT_RG ? 0 : desired;
  p->format = format;
  p->n_groups = int32_t(box.word[kBoxGroups]);
  p->n_slots = box.word[kBoxSlots];
  p->n_heavy = int32_t(box.word[kBoxHeavy]);
  p->nnz = box.word[kBoxNnz];
  p->n_long = box.word[kBoxLong];
  return ARGCSR_OK;
}

constexpr int kMaxDevices = 64;
// Step-1 groups of argcsr_convert_noalloc pass through this host buffer on
// their way to the device (copied and waited for chunk by chunk).
constexpr int32_t kGroupChunk = 1 << 16;
argcsr_group_info g_group_chunk[kGroupChunk];
std::mutex g_noalloc_mu;                    // one argcsr_convert_noalloc at a time
void* g_noalloc_ptr[kMaxDevices] = {};       // device address of `scratch`, per device

// The current device's address of `scratch` (looked up once per device,
// with that device current).  Caller holds g_noalloc_mu.
int noalloc_scratch(void** out) {
  int dev = -1;
  ARGCSR_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(ARGCSR_EUNSUPPORTED, "device %d", dev);
  if (!g_noalloc_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(ARGCSR_EHIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    g_noalloc_ptr[dev] = p;
  }
  *out = g_noalloc_ptr[dev];
  return ARGCSR_OK;
}

// All four steps.  With `fixed` (argcsr_convert_noalloc) the scratch is the
// given device memory of fixed_bytes, step 1 runs on the host from
// row_ptr_host (required) and its groups reach the device through
// g_group_chunk; nothing is allocated.
int convert_impl(int32_t n_rows, int32_t n_cols, const int32_t* row_ptr_host,
                 const int32_t* row_ptr, const int32_t* col, const double* val,
                 argcsr_matrix* out, hipStream_t s, bool fixed,
                 const argcsr_device_plan* planned = nullptr,
                 const argcsr_group_info* pregrouped = nullptr) {
  if (!out) return fail(ARGCSR_EINVAL, "out is NULL");
  if (n_rows < 0 || n_cols < 0) return fail(ARGCSR_EINVAL, "negative dimension");
  if (out->n_rows != n_rows || out->n_cols != n_cols)
    return fail(ARGCSR_EINVAL, "out->n_rows/n_cols do not match the arguments");
  const int32_t T = out->block_dim;
  if (T < 1 || T > kMaxBlockDim)
    return fail(ARGCSR_EUNSUPPORTED, "block_dim %d outside [1, %d]", T, kMaxBlockDim);
  if (out->format != ARGCSR_FORMAT_ARG && out->format != ARGCSR_FORMAT_RG)
    return fail(ARGCSR_EINVAL, "unknown format %d", out->format);
  if (out->format == ARGCSR_FORMAT_ARG && out->desired_chunk_size < 1 && !out->region_desired)
    return fail(ARGCSR_EINVAL, "desired_chunk_size < 1");
  if (out->dtype < ARGCSR_F64 || out->dtype > ARGCSR_F16)
    return fail(ARGCSR_EINVAL, "unknown dtype %d", out->dtype);
  if (out->n_groups < 0 || out->n_slots < 0) return fail(ARGCSR_EINVAL, "negative size in out");
  const int32_t* regions = out->format == ARGCSR_FORMAT_ARG ? out->region_desired : nullptr;
  int rc = check_regions(n_rows, out->region_rows, regions);
  if (rc) return rc;
  void* fixed_ptr = nullptr;
  if (fixed) {
    if (!row_ptr_host)
      return fail(ARGCSR_EINVAL, "argcsr_convert_noalloc needs row_ptr_host (step 1 on the host)");
    // the documented limit: 24 bytes, 16 a thousand groups, the long-row list
    const size_t need = 24 + 16 * ((size_t(out->n_groups) + 1023) / 1024) +
                        2 * sizeof(int32_t) * size_t(long_capacity(out->n_slots, T));
    if (need > kNoAllocScratchBytes)
      return fail(ARGCSR_EINVAL,
                  "the conversion needs %zu bytes of scratch, more than the %zu bytes "
                  "argcsr_convert_noalloc holds", need, kNoAllocScratchBytes);
  }
  // step 1: on the host from row_ptr_host, or on the device (group.hip)
  std::vector<argcsr_group_info> host_groups;
  argcsr_device_plan own_plan;
  int64_t nnz = 0;
  int32_t G = 0;
  bool groups_uploaded = false;
  if (n_rows > 0 && !row_ptr && !row_ptr_host) return fail(ARGCSR_EINVAL, "row_ptr is NULL");
  if (planned && n_rows > 0 && !row_ptr) return fail(ARGCSR_EINVAL, "row_ptr is NULL");
  if (!planned && !row_ptr_host) {
    if (n_rows > 0) {
      rc = build_plan(n_rows, row_ptr, T, out->desired_chunk_size, out->format, out->region_rows,
                      regions, s, &own_plan);
      if (rc) return rc;
    }
    planned = &own_plan;
  }
  if (planned) {
    // steps 1-3 are done (here or by argcsr_plan_device_keep)
    G = planned->n_groups;
    nnz = planned->nnz;
  } else if (row_ptr_host && pregrouped) {
    // step 1 done (and row_ptr_host validated) by the caller
    nnz = n_rows > 0 ? row_ptr_host[n_rows] : 0;
    G = out->n_groups;
    if (G > 0 && !out->groups) return fail(ARGCSR_EINVAL, "NULL device buffer");
    if (G > 0)
      ARGCSR_HIP(hipMemcpyAsync(out->groups, pregrouped, sizeof(argcsr_group_info) * size_t(G),
                                hipMemcpyHostToDevice, s));
    groups_uploaded = true;
  } else if (row_ptr_host) {
    rc = check_row_ptr(n_rows, row_ptr_host);
    if (rc) return rc;
    nnz = n_rows > 0 ? row_ptr_host[n_rows] : 0;
    if (fixed) {
      if (out->n_groups > 0 && !out->groups) return fail(ARGCSR_EINVAL, "NULL device buffer");
      rc = noalloc_scratch(&fixed_ptr);
      if (rc) return rc;
      // groups go to out->groups a chunk at a time, never past out->n_groups
      int32_t filled = 0;
      auto flush = [&]() -> int {
        if (filled == 0) return ARGCSR_OK;
        ARGCSR_HIP(hipMemcpyAsync(out->groups + (G - filled), g_group_chunk,
                                  sizeof(argcsr_group_info) * size_t(filled),
                                  hipMemcpyHostToDevice, s));
        ARGCSR_HIP(hipStreamSynchronize(s));       // the buffer is reused next
        filled = 0;
        return ARGCSR_OK;
      };
      rc = for_each_group(n_rows, row_ptr_host, T, out->desired_chunk_size, out->format,
                          out->region_rows, regions, [&](int32_t first, int32_t size) -> int {
                            if (G >= out->n_groups)
                              return fail(ARGCSR_EINVAL, "out->n_groups = %d but the matrix "
                                          "has more groups", out->n_groups);
                            g_group_chunk[filled++] = argcsr_group_info{first, size, 0, 0};
                            ++G;
                            return filled == kGroupChunk ? flush() : 0;
                          });
      if (rc) return rc;
      rc = flush();
      if (rc) return rc;
      groups_uploaded = true;
    } else {
      rc = group_rows(n_rows, row_ptr_host, T, out->desired_chunk_size, out->format,
                      &host_groups, out->region_rows, regions);
      if (rc) return rc;
      G = (int32_t)host_groups.size();
    }
  }
  if (G != out->n_groups)
    return fail(ARGCSR_EINVAL, "out->n_groups = %d but the matrix has %d groups", out->n_groups, G);
  out->nnz = nnz;
  out->heavy_chunk = heavy_chunk_for(T, out->n_slots, G);
  if (G == 0) {
    out->n_heavy = 0;
    if (out->n_slots != 0) return fail(ARGCSR_EINVAL, "out->n_slots must be 0 for an empty matrix");
    return ARGCSR_OK;
  }
  if (!row_ptr || !out->groups || !out->threads_mapping || !out->columns || !out->values ||
      (nnz > 0 && (!col || !val)))
    return fail(ARGCSR_EINVAL, "NULL device buffer");

  DeviceScratch ws;
  void* base = fixed_ptr;
  if (!fixed) {
    rc = ws.alloc(convert_scratch(out->n_slots, T), s);
    if (rc) return rc;
    base = ws.ptr();
  }
  auto* st = static_cast<Status*>(base);
  auto* share_slots = reinterpret_cast<int64_t*>(static_cast<char*>(base) + kHeadBytes);
  const int64_t* heavy_parts = share_slots + kChunkBlocks;
  // (group, first step) per tile of the fill's long blocks
  int2* long_list = reinterpret_cast<int2*>(share_slots + kChunkBlocks + 2 * kScanBlocks);
  ResultBox box;
  rc = box.init(fixed ? reinterpret_cast<int64_t*>(st + 1) : nullptr, s);
  if (rc) return rc;
  // uses the caller's slot count; it is checked against the device total
  // before anything is written to the caller's heavy_groups buffer
  const int32_t heavy_chunk = out->heavy_chunk;
  int64_t slots = 0, heavy = 0, n_long = 0;

  if (planned) {
    slots = planned->n_slots;
    heavy = planned->n_heavy;
    n_long = planned->n_long;
  } else {
    clear_words_kernel<<<1, 64, 0, s>>>(static_cast<int32_t*>(base),
                                        int32_t(kHeadBytes / sizeof(int32_t)));
    if (!groups_uploaded)
      ARGCSR_HIP(hipMemcpyAsync(out->groups, host_groups.data(),
                                sizeof(argcsr_group_info) * size_t(G), hipMemcpyHostToDevice, s));
    launch_chunks(row_ptr, out->groups, G, nullptr, T, out->format, out->threads_mapping,
                  share_slots, s);
    int64_t* parts = share_slots + kChunkBlocks;
    offsets_kernel<<<kScanBlocks, kScanBlock, 0, s>>>(out->groups, G, nullptr, T, share_slots,
                                                      parts, parts + kScanBlocks, st, row_ptr,
                                                      n_rows, box.dev);
    ARGCSR_HIP(hipGetLastError());
    rc = box.read(s);
    if (rc) return rc;
    slots = box.word[kBoxSlots];
    heavy = box.word[kBoxHeavy];
    n_long = box.word[kBoxLong];
  }
  if (slots > INT32_MAX)
    return fail(ARGCSR_EOVERFLOW, "%lld slots exceed INT32_MAX", (long long)slots);
  if (slots != out->n_slots)
    return fail(ARGCSR_EINVAL, "out->n_slots = %lld but the matrix needs %lld",
                (long long)out->n_slots, (long long)slots);
  if (out->heavy_groups && heavy != out->n_heavy)
    return fail(ARGCSR_EINVAL, "out->n_heavy = %d but the matrix has %lld heavy groups",
                out->n_heavy, (long long)heavy);
  out->n_heavy = int32_t(heavy);
  if (planned) {
    heavy_parts = planned->heavy_parts;
    const int64_t blocks = std::min<int64_t>((4 * int64_t(G) + n_rows + 255) / 256, 2048);
    adopt_plan_kernel<<<dim3(uint32_t(blocks)), 256, 0, s>>>(
        reinterpret_cast<const int32_t*>(planned->groups), 4 * int64_t(G), planned->tm, n_rows,
        reinterpret_cast<int32_t*>(out->groups), out->threads_mapping);
  }
  const int32_t stage = fill_stage(T, out->n_slots, G);
  if ((out->heavy_groups && out->n_heavy > 0) || n_long > 0)
    schedule_kernel<<<kScanBlocks, kScanBlock, 0, s>>>(
        out->groups, G, heavy_chunk, stage, heavy_parts, heavy_parts + kScanBlocks,
        out->n_heavy > 0 ? out->heavy_groups : nullptr, long_list);

  switch (out->dtype) {
    case ARGCSR_F64:
      launch_fill<ARGCSR_F64>(s, row_ptr, col, val, stage, box.dev, long_list, int32_t(n_long), out);
      break;
    case ARGCSR_F32:
      launch_fill<ARGCSR_F32>(s, row_ptr, col, val, stage, box.dev, long_list, int32_t(n_long), out);
      break;
    case ARGCSR_BF16:
      launch_fill<ARGCSR_BF16>(s, row_ptr, col, val, stage, box.dev, long_list, int32_t(n_long), out);
      break;
    default:
      launch_fill<ARGCSR_F16>(s, row_ptr, col, val, stage, box.dev, long_list, int32_t(n_long), out);
      break;
  }
  ARGCSR_HIP(hipGetLastError());
  rc = box.read(s);
  if (rc) return rc;
  ws.idle();
  box.idle();
  if (box.word[kBoxBadColumn])
    return fail(ARGCSR_EINVAL, "a column index lies outside [0, %d)", n_cols);
  return ARGCSR_OK;
}

}  // namespace
}  // namespace argcsr

namespace argcsr {

int convert_pregrouped(int32_t n_rows, int32_t n_cols, const int32_t* row_ptr_host,
                       const argcsr_group_info* groups_host, const int32_t* row_ptr,
                       const int32_t* col, const double* val, argcsr_matrix* out,
                       hipStream_t s) {
  if (!row_ptr_host || (out && out->n_groups > 0 && !groups_host))
    return fail(ARGCSR_EINVAL, "a pregrouped conversion needs row_ptr_host and the groups");
  return convert_impl(n_rows, n_cols, row_ptr_host, row_ptr, col, val, out, s, false, nullptr,
                      groups_host);
}

}  // namespace argcsr

extern "C" int argcsr_convert(int32_t n_rows, int32_t n_cols, const int32_t* row_ptr_host,
                              const int32_t* row_ptr, const int32_t* col, const double* val,
                              argcsr_matrix* out, void* stream) {
  argcsr::clear_error();
  return argcsr::convert_impl(n_rows, n_cols, row_ptr_host, row_ptr, col, val, out,
                              static_cast<hipStream_t>(stream), false);
}

extern "C" int argcsr_convert_noalloc(int32_t n_rows, int32_t n_cols, const int32_t* row_ptr_host,
                                      const int32_t* row_ptr, const int32_t* col,
                                      const double* val, argcsr_matrix* out, void* stream) {
  argcsr::clear_error();
  std::lock_guard<std::mutex> lock(argcsr::g_noalloc_mu);
  return argcsr::convert_impl(n_rows, n_cols, row_ptr_host, row_ptr, col, val, out,
                              static_cast<hipStream_t>(stream), true);
}

namespace argcsr {
namespace {

// Steps 1-3 from a device row_ptr into *p, and the sizes of the result.
int plan_device_impl(int32_t n_rows, const int32_t* row_ptr, int32_t block_dim,
                     int32_t desired_chunk_size, int32_t format, int32_t* n_groups,
                     int64_t* n_slots, int32_t* n_heavy, hipStream_t s, argcsr_device_plan* p,
                     const int32_t* row_ptr_host = nullptr) {
  if (!n_groups || !n_slots) return fail(ARGCSR_EINVAL, "NULL output pointer");
  if (n_rows < 0) return fail(ARGCSR_EINVAL, "n_rows < 0");
  if (format != ARGCSR_FORMAT_ARG && format != ARGCSR_FORMAT_RG)
    return fail(ARGCSR_EINVAL, "unknown format %d", format);
  if (block_dim < 1 || block_dim > kMaxBlockDim ||
      (format == ARGCSR_FORMAT_ARG && desired_chunk_size < 1))
    return fail(ARGCSR_EINVAL, "block_dim must be in [1, %d] and desired_chunk_size >= 1",
                kMaxBlockDim);
  if (n_rows > 0 && !row_ptr) return fail(ARGCSR_EINVAL, "row_ptr is NULL");
  if (n_rows > 0) {
    const int rc = build_plan(n_rows, row_ptr, block_dim, desired_chunk_size, format, 0, nullptr,
                              s, p, row_ptr_host);
    if (rc) return rc;
  }
  *n_groups = p->n_groups;
  *n_slots = p->n_slots;
  if (n_heavy) *n_heavy = p->n_heavy;
  if (p->n_slots > INT32_MAX)
    return fail(ARGCSR_EOVERFLOW, "%lld slots exceed INT32_MAX", (long long)p->n_slots);
  return ARGCSR_OK;
}

}  // namespace
}  // namespace argcsr

extern "C" int argcsr_plan_device(int32_t n_rows, const int32_t* row_ptr, int32_t block_dim,
                                  int32_t desired_chunk_size, int32_t format, int32_t* n_groups,
                                  int64_t* n_slots, int32_t* n_heavy, void* stream) {
  argcsr::clear_error();
  argcsr_device_plan p;
  return argcsr::plan_device_impl(n_rows, row_ptr, block_dim, desired_chunk_size, format,
                                  n_groups, n_slots, n_heavy, static_cast<hipStream_t>(stream),
                                  &p);
}

namespace argcsr {
namespace {

int plan_keep_impl(int32_t n_rows, const int32_t* row_ptr_host, const int32_t* row_ptr,
                   int32_t block_dim, int32_t desired_chunk_size, int32_t format,
                   int32_t* n_groups, int64_t* n_slots, int32_t* n_heavy,
                   argcsr_device_plan** plan, hipStream_t s) {
  if (!plan) return fail(ARGCSR_EINVAL, "plan is NULL");
  *plan = nullptr;
  auto* p = new (std::nothrow) argcsr_device_plan();
  if (!p) return fail(ARGCSR_ENOMEM, "device plan");
  p->n_rows = n_rows;
  p->block_dim = block_dim;
  p->desired_chunk_size = format == ARGCSR_FORMAT_RG ? 0 : desired_chunk_size;
  p->format = format;
  const int rc = plan_device_impl(n_rows, row_ptr, block_dim, desired_chunk_size, format,
                                  n_groups, n_slots, n_heavy, s, p, row_ptr_host);
  if (rc) {
    delete p;
    return rc;
  }
  *plan = p;
  return ARGCSR_OK;
}

}  // namespace
}  // namespace argcsr

extern "C" int argcsr_plan_device_keep(int32_t n_rows, const int32_t* row_ptr, int32_t block_dim,
                                       int32_t desired_chunk_size, int32_t format,
                                       int32_t* n_groups, int64_t* n_slots, int32_t* n_heavy,
                                       argcsr_device_plan** plan, void* stream) {
  argcsr::clear_error();
  return argcsr::plan_keep_impl(n_rows, nullptr, row_ptr, block_dim, desired_chunk_size, format,
                                n_groups, n_slots, n_heavy, plan,
                                static_cast<hipStream_t>(stream));
}

extern "C" int argcsr_plan_keep(int32_t n_rows, const int32_t* row_ptr_host,
                                const int32_t* row_ptr, int32_t block_dim,
                                int32_t desired_chunk_size, int32_t format, int32_t* n_groups,
                                int64_t* n_slots, int32_t* n_heavy, argcsr_device_plan** plan,
                                void* stream) {
  using namespace argcsr;
  clear_error();
  if (n_rows > 0 && !row_ptr_host) {
    if (plan) *plan = nullptr;
    return fail(ARGCSR_EINVAL, "row_ptr_host is NULL");
  }
  return plan_keep_impl(n_rows, row_ptr_host, row_ptr, block_dim, desired_chunk_size, format,
                        n_groups, n_slots, n_heavy, plan, static_cast<hipStream_t>(stream));
}

extern "C" int argcsr_convert_planned(const argcsr_device_plan* plan, int32_t n_cols,
                                      const int32_t* row_ptr, const int32_t* col,
                                      const double* val, argcsr_matrix* out, void* stream) {
  using namespace argcsr;
  clear_error();
  if (!plan || !out) return fail(ARGCSR_EINVAL, "plan or out is NULL");
  if (out->n_rows != plan->n_rows || out->block_dim != plan->block_dim ||
      out->format != plan->format || out->n_groups != plan->n_groups ||
      out->n_slots != plan->n_slots ||
      (plan->format == ARGCSR_FORMAT_ARG && out->desired_chunk_size != plan->desired_chunk_size))
    return fail(ARGCSR_EINVAL, "out does not describe the planned matrix");
  if (out->region_desired) return fail(ARGCSR_EINVAL, "a device plan has one desired_chunk_size");
  if (out->heavy_groups && out->n_heavy != plan->n_heavy)
    return fail(ARGCSR_EINVAL, "out->n_heavy = %d but the plan has %d", out->n_heavy,
                plan->n_heavy);
  return convert_impl(plan->n_rows, n_cols, nullptr, row_ptr, col, val, out,
                      static_cast<hipStream_t>(stream), false, plan);
}

extern "C" int argcsr_device_plan_destroy(argcsr_device_plan* plan) {
  delete plan;
  return ARGCSR_OK;
}
