// Conversion step 1 (grouping, Sec. 3) on the GPU.
//
// The rule is the host's (plan.cpp): from a group's first row s the group
// takes rows while it keeps at most block_dim rows and at most
// desired*block_dim nonzeros, and always takes row s.  So the group opened
// at s ends at
//   next(s) = max(s+1, max{e <= min(n, s+block_dim) : rp[e] - rp[s] <= budget}),
// a function of s alone, and the groups are the path 0 -> next(0) ->
// next(next(0)) -> ... -> n.  Walking it is sequential; here the rows are cut
// into blocks of kGroupRows, and because a group takes at most block_dim
// rows, the path enters a block within its first block_dim rows whatever
// came before:
//   1. group_map_kernel    per block and for each of those block_dim entry
//                          rows: where the path from it enters the next block
//                          and how many groups it opens on the way (pointer
//                          doubling in LDS);
//   2. group_entry_kernel  one workgroup composes the blocks' maps: the
//                          entry row of every block and the groups before it;
//   3. group_emit_kernel   per block: the rows the path visits from the
//                          block's entry row (doubling again, marking), which
//                          are its groups.
// The result is the host scan's, row for row.
//
// What bounds it: three launches of latency chains; the bytes are few (4 a
// row read, 2 a row written and read again).  Measured on MI355X on the
// power-law matrix of 10^6 rows (T = 64, 63 517 groups): 15 + 7.4 + 11.8 us.
// Jump tables over all rows (binary lifting: 10 launches, 84 bytes a row
// written) took 75 us.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "group.hpp"

namespace argcsr {
namespace {

constexpr int kGroupBlock = 1024;                      // threads
constexpr int kRowsPer = kGroupRows / kGroupBlock;     // rows a thread handles
constexpr int kMaxGroupDim = 1024;   // block_dim limit of plan/convert
constexpr int kEntryBlock = 1024;    // threads of group_entry_kernel
constexpr int kEntryMaps = 28672;    // map entries it holds in LDS at a time
constexpr int kEntryBlocks = 1024;   // blocks it takes at a time, at most

// A path segment of one block: groups opened (high half) and the row it
// leads to (low half), local to the block or to the next one.
__device__ __forceinline__ uint32_t pack_path(uint32_t groups, uint32_t row) {
  return groups << 16 | row;
}

// Step 1.1, and the row_ptr validation (rp[0] == 0, non-decreasing).
// steps[r] = next(r) - r (at most 1024) is kept for step 1.3.  Doubling runs
// in place: a row's word is one 32-bit value that always says "this many
// groups lead to that row", so reading another row's word before or after
// its update only changes how soon the loop ends, not what it ends with.
__global__ __launch_bounds__(kGroupBlock) void group_map_kernel(
    int32_t n, const int32_t* __restrict__ rp, int32_t block_dim, int64_t budget,
    int32_t region_rows, const int32_t* __restrict__ region_desired,
    uint16_t* __restrict__ steps, uint32_t* __restrict__ maps, int32_t* __restrict__ bad_blocks) {
  __shared__ int32_t srp[kGroupRows + kMaxGroupDim + 1];
  __shared__ uint32_t path[kGroupRows];
  const int64_t base = int64_t(blockIdx.x) * kGroupRows;
  const int32_t limit = int32_t(min(int64_t(kGroupRows), int64_t(n) - base));   // rows of the block
  const int32_t span = int32_t(min(int64_t(n) - base, int64_t(kGroupRows) + block_dim));
  for (int32_t i = threadIdx.x; i <= span; i += kGroupBlock) srp[i] = rp[base + i];
  __syncthreads();
  // next(l): the largest e in [l, top] with srp[e] <= most, at least l + 1;
  // the rows of a thread are searched together, step by step
  int bad = 0;
  int32_t at[kRowsPer], top[kRowsPer];
  int64_t most[kRowsPer];
#pragma unroll
  for (int k = 0; k < kRowsPer; ++k) {
    const int32_t l = k * kGroupBlock + int32_t(threadIdx.x);
    at[k] = l;
    top[k] = l < limit ? min(span, l + block_dim) : l;
    most[k] = 0;
    if (l >= limit) continue;
    // a per-region desiredChunkSize: the region of the group's first row
    most[k] = int64_t(srp[l]) + (region_desired
                                     ? int64_t(region_desired[(base + l) / region_rows]) * block_dim
                                     : budget);
    if (srp[l + 1] < srp[l] || (base + l == 0 && srp[0] != 0)) {
      bad = 1;
      top[k] = l;                         // a malformed row opens a group of its own
    }
  }
  for (int32_t step = 1 << (31 - __clz(block_dim)); step > 0; step >>= 1) {
#pragma unroll
    for (int k = 0; k < kRowsPer; ++k)
      if (at[k] + step <= top[k] && int64_t(srp[at[k] + step]) <= most[k]) at[k] += step;
  }
#pragma unroll
  for (int k = 0; k < kRowsPer; ++k) {
    const int32_t l = k * kGroupBlock + int32_t(threadIdx.x);
    if (l >= limit) continue;
    const int32_t e = max(at[k], l + 1);
    steps[base + l] = uint16_t(e - l);
    path[l] = pack_path(1, uint32_t(e));
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) bad_blocks[blockIdx.x] = bad;
  int more = 1;
  while (__syncthreads_or(more)) {
    more = 0;
#pragma unroll
    for (int k = 0; k < kRowsPer; ++k) {
      const int32_t l = k * kGroupBlock + int32_t(threadIdx.x);
      if (l >= limit) continue;
      const uint32_t p = path[l];
      if (int32_t(p & 0xffffu) < limit) {
        const uint32_t q = path[p & 0xffffu];
        path[l] = pack_path((p >> 16) + (q >> 16), q & 0xffffu);
        more |= int32_t(q & 0xffffu) < limit;
      }
    }
  }
  // entry rows past a short last block: the path has ended (row n is local
  // row `limit`, the next block's row 0)
  for (int32_t e = threadIdx.x; e < block_dim; e += kGroupBlock) {
    const uint32_t p = e < limit ? path[e] : pack_path(0, uint32_t(e));
    maps[int64_t(blockIdx.x) * block_dim + e] = pack_path(p >> 16, (p & 0xffffu) - uint32_t(limit));
  }
}

// Step 1.2, one workgroup.  The maps of up to kEntryMaps / block_dim blocks
// are held in LDS at a time; the blocks are cut into 1024 / block_dim
// segments, every (segment, entry row) walks its segment's maps, one thread
// walks the segments, then one thread a segment walks its blocks again from
// the now known entry row: 2 * blocks / segments + segments dependent LDS
// reads instead of one per block.
__global__ __launch_bounds__(kEntryBlock) void group_entry_kernel(
    int32_t n_blocks, int32_t block_dim, const uint32_t* __restrict__ maps,
    int2* __restrict__ entries, const int32_t* __restrict__ bad_blocks,
    GroupCount* __restrict__ count,
    int32_t* __restrict__ clear, int64_t clear_words) {
  __shared__ uint16_t exits[kEntryMaps];
  __shared__ uint16_t seg_map[kEntryBlock];
  __shared__ uint16_t seg_entry[kEntryBlock];
  __shared__ uint16_t entry_of[kEntryBlocks];
  __shared__ int wave_tot[kEntryBlock / 64];
  __shared__ int entry_next;
  const int tid = int(threadIdx.x);
  for (int64_t i = tid; i < clear_words; i += kEntryBlock) clear[i] = 0;
  const int32_t at_a_time = min(kEntryBlocks, kEntryMaps / block_dim);
  const int32_t segs = kEntryBlock / block_dim;
  int32_t entry = 0, before = 0;                 // of the first block of the round
  for (int32_t b0 = 0; b0 < n_blocks; b0 += at_a_time) {
    const int32_t nb = min(at_a_time, n_blocks - b0);
    const uint32_t* m = maps + int64_t(b0) * block_dim;
#pragma unroll 8
    for (int32_t i = tid; i < nb * block_dim; i += kEntryBlock) exits[i] = uint16_t(m[i]);
    __syncthreads();
    const int32_t per = (nb + segs - 1) / segs;
    const int32_t s = tid / block_dim;
    if (s < segs) {
      int32_t e = tid % block_dim;
      for (int32_t b = s * per; b < min(nb, (s + 1) * per); ++b) e = exits[b * block_dim + e];
      seg_map[tid] = uint16_t(e);
    }
    __syncthreads();
    if (tid == 0) {
      int32_t e = entry;
      for (int32_t q = 0; q < segs; ++q) {
        seg_entry[q] = uint16_t(e);
        e = seg_map[q * block_dim + e];
      }
      entry_next = e;
    }
    __syncthreads();
    if (tid < segs) {
      int32_t e = seg_entry[tid];
      for (int32_t b = tid * per; b < min(nb, (tid + 1) * per); ++b) {
        entry_of[b] = uint16_t(e);
        e = exits[b * block_dim + e];
      }
    }
    __syncthreads();
    // groups before each block
    const int32_t e = tid < nb ? entry_of[tid] : 0;
    const int32_t g = tid < nb ? int32_t(m[int64_t(tid) * block_dim + e] >> 16) : 0;
    const int incl = wave_inclusive_scan(g);
    if (lane_id() == 63) wave_tot[tid >> 6] = incl;
    __syncthreads();
    int32_t base = before, all = 0;
    for (int w = 0; w < kEntryBlock / 64; ++w) {
      if (w < (tid >> 6)) base += wave_tot[w];
      all += wave_tot[w];
    }
    if (tid < nb) entries[b0 + tid] = int2{e, base + incl - g};
    before += all;
    entry = entry_next;
    __syncthreads();                             // LDS is reused by the next round
  }
  int bad = 0;
  for (int32_t b = tid; b < n_blocks; b += kEntryBlock) bad |= bad_blocks[b];
  bad = __syncthreads_or(bad);
  if (tid == 0) *count = GroupCount{before, bad};
}

// Step 1.3.  With J = next^(2^k) and the first 2^k rows of the path marked,
// marking J of every marked row gives the first 2^(k+1); J is squared in
// between (read, barrier, write).  It ends when a round marks nothing new.
__global__ __launch_bounds__(kGroupBlock) void group_emit_kernel(
    int32_t n, const uint16_t* __restrict__ steps, const int2* __restrict__ entries,
    argcsr_group_info* __restrict__ groups) {
  __shared__ uint16_t jump[kGroupRows];
  __shared__ __align__(4) uint8_t mark[kGroupRows];
  __shared__ int wave_tot[kGroupBlock / 64];
  static_assert(kRowsPer == 4, "a thread's marks are read as one 4-byte word");
  const int64_t base = int64_t(blockIdx.x) * kGroupRows;
  const int32_t limit = int32_t(min(int64_t(kGroupRows), int64_t(n) - base));
  const int2 in = entries[blockIdx.x];           // entry row, groups before the block
  const int tid = int(threadIdx.x);
  int32_t j[kRowsPer];
#pragma unroll
  for (int k = 0; k < kRowsPer; ++k) {
    const int32_t l = k * kGroupBlock + tid;
    j[k] = l < limit ? l + steps[base + l] : limit;
    jump[l] = uint16_t(j[k]);
    mark[l] = l == in.x && l < limit ? 1 : 0;
  }
  int more = 1;
  while (__syncthreads_or(more)) {
    more = 0;
#pragma unroll
    for (int k = 0; k < kRowsPer; ++k) {
      const int32_t l = k * kGroupBlock + tid;
      if (j[k] < limit) {
        if (mark[l] && !mark[j[k]]) {
          mark[j[k]] = 1;
          more = 1;
        }
        j[k] = jump[j[k]];
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRowsPer; ++k) jump[k * kGroupBlock + tid] = uint16_t(j[k]);
  }
  // rows 4*tid .. 4*tid+3: a group starts at each marked one
  uint32_t mine = *reinterpret_cast<const uint32_t*>(mark + kRowsPer * tid);
  const int own = __popc(mine);
  const int incl = wave_inclusive_scan(own);
  if (lane_id() == 63) wave_tot[tid >> 6] = incl;
  __syncthreads();
  int32_t i = in.y + incl - own;
  for (int w = 0; w < (tid >> 6); ++w) i += wave_tot[w];
  while (mine) {
    const int64_t r = base + kRowsPer * tid + (__builtin_ctz(mine) >> 3);
    mine &= mine - 1;
    groups[i++] = argcsr_group_info{int32_t(r), int32_t(steps[r]), 0, 0};
  }
}

}  // namespace

namespace {

// The work area: maps | entries | regions | bad flags | steps.
struct Work {
  int64_t n_blocks, n_regions;
  size_t entries, regions, bad, steps, bytes;       // byte offsets, and the end
};

Work work_of(int32_t n, int32_t block_dim, int32_t format, int32_t region_rows,
             const int32_t* region_desired) {
  Work w;
  w.n_blocks = (int64_t(n) + kGroupRows - 1) / kGroupRows;
  w.n_regions = region_desired && format != ARGCSR_FORMAT_RG
                    ? (int64_t(n) + region_rows - 1) / region_rows : 0;
  w.entries = (sizeof(uint32_t) * size_t(w.n_blocks) * size_t(block_dim) + 7) & ~size_t(7);
  w.regions = w.entries + sizeof(int2) * size_t(w.n_blocks);
  w.bad = w.regions + sizeof(int32_t) * size_t(w.n_regions);
  w.steps = w.bad + sizeof(int32_t) * size_t(w.n_blocks);
  w.bytes = w.steps + sizeof(uint16_t) * size_t(n);
  return w;
}

}  // namespace

size_t group_work_bytes(int32_t n, int32_t block_dim, int32_t format, int32_t region_rows,
                        const int32_t* region_desired) {
  return work_of(n, block_dim, format, region_rows, region_desired).bytes;
}

int group_on_device(int32_t n, const int32_t* row_ptr, int32_t block_dim, int32_t desired,
                    int32_t format, int32_t region_rows, const int32_t* region_desired,
                    argcsr_group_info* groups, GroupCount* count, int32_t* clear,
                    int64_t clear_words, void* work, hipStream_t s) {
  const bool row_grouped = format == ARGCSR_FORMAT_RG;
  const Work w = work_of(n, block_dim, format, region_rows, region_desired);
  char* p = static_cast<char*>(work);
  auto* maps = reinterpret_cast<uint32_t*>(p);
  auto* entries = reinterpret_cast<int2*>(p + w.entries);
  auto* regions = reinterpret_cast<int32_t*>(p + w.regions);
  auto* bad = reinterpret_cast<int32_t*>(p + w.bad);
  auto* steps = reinterpret_cast<uint16_t*>(p + w.steps);
  const int64_t n_blocks = w.n_blocks;
  if (w.n_regions)
    ARGCSR_HIP(hipMemcpyAsync(regions, region_desired, sizeof(int32_t) * size_t(w.n_regions),
                              hipMemcpyHostToDevice, s));
  group_map_kernel<<<dim3(uint32_t(n_blocks)), kGroupBlock, 0, s>>>(
      n, row_ptr, block_dim, row_grouped ? INT64_MAX / 2 : int64_t(desired) * block_dim,
      region_rows > 0 ? region_rows : 1, w.n_regions ? regions : nullptr, steps, maps, bad);
  group_entry_kernel<<<1, kEntryBlock, 0, s>>>(int32_t(n_blocks), block_dim, maps, entries, bad,
                                               count, clear, clear_words);
  group_emit_kernel<<<dim3(uint32_t(n_blocks)), kGroupBlock, 0, s>>>(n, steps, entries, groups);
  ARGCSR_HIP(hipGetLastError());
  return ARGCSR_OK;
}

}  // namespace argcsr
