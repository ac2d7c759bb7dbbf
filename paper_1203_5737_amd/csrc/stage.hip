// Staging of x for banded matrices: an extension of the ARG-CSR storage.
//
// Sec. 4 stages in shared memory the data a block of threads reuses.  In a
// banded matrix the rows of a group name a few runs of consecutive columns
// (for a stencil: the grid lines around the group's own), so the part of x a
// group reads is small and can be staged the same way.  Per group, the
// distinct columns its slots name are merged into windows (two neighbouring
// columns stay in one window when at most `gap` columns between them are
// absent), and every window is cut into tiles of 64 consecutive columns
// (the last one shorter).  A slot then stores, instead of its column, a
// 16-bit position in its group's staged tiles: 64*q + (column - start of
// tile q), 0xFFFF for an artificial zero.  The SpMV loads a group's tiles
// into LDS with coalesced loads and reads x from there; the index stream is
// 2 bytes per slot instead of 4.
//
//   stage_kernel<false>  per group: its tile count (written to tile_ptr[g+1],
//                        a negative code for a group that cannot be staged)
//   stage_scan_kernel    tile_ptr as an exclusive scan, the total and the
//                        largest group's count
//   stage_kernel<true>   per group: its tiles (first column, length) and the
//                        position of every slot
//
// One workgroup of one, two or four waves per group.  The group's columns are marked in
// a bitmap in LDS (offset by the group's smallest column), a segment of it at
// a time; the windows follow from the distances between consecutive set bits,
// which each thread finds over its own range of bitmap words with the last
// set bit of the threads before it.
#include <hip/hip_runtime.h>

#include <climits>

#include "common.hpp"
#include "mailbox.hpp"
#include "stage.hpp"

namespace argcsr {
namespace {

constexpr int kSegBits = 1 << 15;         // columns marked at a time: 4 KB of LDS
constexpr int kSegWords = kSegBits / 32;
constexpr int kHeldSlots = 16;            // slots a thread holds in registers
constexpr int kNoSpan = -1;               // tile_ptr codes of the count pass
constexpr int kNoTiles = -2;

// words of the result slot
constexpr int kBoxTotal = 0, kBoxMaxTiles = 1, kBoxUnstageable = 2, kBoxMismatch = 3;

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef uint16_t v4u16 __attribute__((ext_vector_type(4)));

// Workgroup-wide reductions and scans over NT threads (NT/64 waves).  `red`
// holds one int per wave; every thread calls, and the call ends with a
// barrier, so `red` is free again.
template <int NT>
__device__ __forceinline__ int block_max(int v, int* red) {
  v = wave_max(v);
  if constexpr (NT == 64) return v;
  if (lane_id() == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) v = red[w] > v ? red[w] : v;
  __syncthreads();
  return v;
}

template <int NT>
__device__ __forceinline__ void block_min_max(int& mn, int& mx, int* red) {
  mx = wave_max(mx);
  mn = INT_MAX - wave_max(INT_MAX - mn);
  if constexpr (NT == 64) return;
  constexpr int kW = NT / 64;
  if (lane_id() == 0) {
    red[threadIdx.x >> 6] = mx;
    red[kW + (threadIdx.x >> 6)] = mn;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    mx = red[w] > mx ? red[w] : mx;
    mn = red[kW + w] < mn ? red[kW + w] : mn;
  }
  // no barrier: the next use of red follows the clearing of the bitmap
}

// The largest v of the threads before this one (-1 if none) and of all.
template <int NT>
__device__ __forceinline__ int block_excl_max(int v, int* red, int* all) {
  const int lane = lane_id();
  const int incl = wave_inclusive_max(v);
  int before = __shfl_up(incl, 1, 64);
  if (lane == 0) before = -1;
  if constexpr (NT == 64) {
    *all = __shfl(incl, 63, 64);
    return before;
  }
  const int wv = int(threadIdx.x >> 6);
  if (lane == 63) red[wv] = incl;
  __syncthreads();
  int m = -1;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wv) before = red[w] > before ? red[w] : before;
    m = red[w] > m ? red[w] : m;
  }
  __syncthreads();
  *all = m;
  return before;
}

// The sum of v over the threads before this one, and over all.
template <int NT>
__device__ __forceinline__ int block_excl_sum(int v, int* red, int* all) {
  const int incl = wave_inclusive_scan(v);
  if constexpr (NT == 64) {
    *all = __shfl(incl, 63, 64);
    return incl - v;
  }
  const int wv = int(threadIdx.x >> 6);
  if (lane_id() == 63) red[wv] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wv) before += red[w];
    total += red[w];
  }
  __syncthreads();
  *all = total;
  return before + incl - v;
}

// Calls f(window start, set bit before it) for every window that starts in
// word w of the bitmap (word bits b, `prev` the last set bit before the word,
// -1 if none): a set bit whose predecessor lies more than gap + 1 columns
// back.  Only the starts of runs of set bits can be one.
template <typename F>
__device__ __forceinline__ void window_starts(uint32_t b, int bit0, int prev, int gap, F f) {
  const uint32_t carry = prev >= 0 && prev == bit0 - 1 ? 1u : 0u;
  uint32_t runs = b & ~((b << 1) | carry);
  while (runs) {
    const int i = __builtin_ctz(runs);
    runs &= runs - 1;
    const uint32_t below = b & ((1u << i) - 1u);
    const int pv = below ? bit0 + 31 - __clz(int(below)) : prev;
    const int p = bit0 + i;
    if (pv < 0 || int64_t(p) - pv - 1 > int64_t(gap)) f(p, pv);
  }
}

// What takes the time: reading the columns (4 bytes a slot), marking, scans and
// lookup, and writing the positions (2 bytes a slot); the group's chain is
// hidden by the other groups of a CU.  The vector ALU issues for 26 of the
// count pass's 36 us (514 instructions a wave) and 40 of the fill pass's 58
// (790), yet fewer instructions per marked column took the same time: neither
// issue nor the stream alone is the bound.  The fill finds the windows again
// that the count found, which nothing carries over.  A
// thread holds up to kHeldSlots columns in registers, so a group that fits
// its workgroup's registers is read once; a longer one is read again (from
// L2) in each of the three phases.  The bitmap covers 2^15 columns at a time
// (a span beyond that takes more rounds of marking), which keeps the LDS of a
// workgroup near 5 KB and the CU full of waves.  Measured on MI355X on the
// 100^3 27-point stencil (T = 128: 7813 groups of 3424 slots): 36 us the count
// pass (3.0 TB/s) and 58 us the fill pass (2.8 TB/s), against 690 and 815 us
// of a kernel with one wave per group, a 32-KB bitmap and slots read one at
// a time in each phase.  One atomic for a thread's four columns instead of
// one each, and the window search skipped inside a window, gave 13% each.
template <bool FILL, int NT>
__global__ __launch_bounds__(NT) void stage_kernel(
    const argcsr_group_info* __restrict__ groups, int32_t n_groups, int32_t T,
    const int32_t* __restrict__ columns, int32_t gap, int32_t* __restrict__ tile_ptr,
    int32_t n_stage_tiles, int32_t* __restrict__ tile_start, int32_t* __restrict__ tile_len,
    uint16_t* __restrict__ local, int64_t* __restrict__ box) {
  constexpr int kVecs = kHeldSlots / 4;
  constexpr int kRound = NT * kHeldSlots;           // slots one round of loads covers
  __shared__ uint32_t bm[kSegWords];
  __shared__ int32_t win_start[kStageMaxTiles];     // relative to the smallest column
  __shared__ int32_t win_prev[kStageMaxTiles];      // the set bit before it (-1 for the first)
  __shared__ int32_t win_base[kStageMaxTiles];      // position of a column minus the column
  __shared__ int red[2 * (NT / 64)];
  __shared__ int tiles_all;
  const int g = int(blockIdx.x);
  if (g >= n_groups) return;
  const int tid = int(threadIdx.x);
  const argcsr_group_info gi = groups[g];
  const int64_t slots = int64_t(gi.chunk_size) * T;
  const int32_t* cb = columns + gi.offset;
  // 16-byte loads (and 8-byte stores) where the group's slots allow them
  const bool vec = ((reinterpret_cast<uintptr_t>(cb) & 15) |
                    (FILL ? reinterpret_cast<uintptr_t>(local + gi.offset) & 7 : 0) |
                    uintptr_t(slots & 3)) == 0;
  const bool held = slots <= kRound;

  // slots 4 * (tid + k * NT) + {0..3} of a round, -1 past the end
  v4i c[kVecs];
  auto load = [&](int64_t base) {
#pragma unroll
    for (int k = 0; k < kVecs; ++k) {
      const int64_t s = base + 4 * int64_t(tid + k * NT);
      c[k] = v4i{-1, -1, -1, -1};
      if (vec) {
        if (s < slots) c[k] = *reinterpret_cast<const v4i*>(cb + s);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (s + e < slots) c[k][e] = cb[s + e];
      }
    }
  };

  // the group's smallest and largest column
  int mn = INT_MAX, mx = -1;
  for (int64_t base = 0; base < slots; base += kRound) {
    load(base);
#pragma unroll
    for (int k = 0; k < kVecs; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = c[k][e];
        if (v >= 0) {
          mn = v < mn ? v : mn;
          mx = v > mx ? v : mx;
        }
      }
    }
  }
  block_min_max<NT>(mn, mx, red);

  int n_win = 0, n_tiles = 0, code = 0;
  if (mx >= 0) {
    const int64_t span = int64_t(mx) - mn + 1;
    if (span > kStageSpanBits) {
      code = kNoSpan;
    } else {
      int prev_seg = -1;                            // last set bit of the segments before
      for (int seg0 = 0; seg0 < int(span); seg0 += kSegBits) {
        const int bits = int(span) - seg0 < kSegBits ? int(span) - seg0 : kSegBits;
        const int nw = (bits + 31) / 32;
        for (int w = tid; w < nw; w += NT) bm[w] = 0u;
        __syncthreads();
        for (int64_t base = 0; base < slots; base += kRound) {
          if (!held) load(base);
#pragma unroll
          for (int k = 0; k < kVecs; ++k) {
            // four neighbouring chunks name neighbouring columns in a banded
            // matrix: bits of one word are set with one atomic
            uint32_t word = 0, bits_of = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const uint32_t r = uint32_t(c[k][e] - mn - seg0);
              const bool in = c[k][e] >= 0 && r < uint32_t(bits);
              if (in && (r >> 5) != word && bits_of) {
                atomicOr(&bm[word], bits_of);
                bits_of = 0;
              }
              if (in) {
                word = r >> 5;
                bits_of |= 1u << (r & 31);
              }
            }
            if (bits_of) atomicOr(&bm[word], bits_of);
          }
        }
        __syncthreads();
        // this thread's words [lo, hi)
        const int per = (nw + NT - 1) / NT;
        const int lo = tid * per < nw ? tid * per : nw;
        const int hi = lo + per < nw ? lo + per : nw;
        int last = -1;
        for (int w = lo; w < hi; ++w) {
          const uint32_t b = bm[w];
          if (b) last = seg0 + 32 * w + 31 - __clz(int(b));
        }
        int last_seg;
        int before = block_excl_max<NT>(last, red, &last_seg);
        if (before < 0) before = prev_seg;
        int starts = 0, prev = before;
        for (int w = lo; w < hi; ++w) {
          const uint32_t b = bm[w];
          window_starts(b, seg0 + 32 * w, prev, gap, [&](int, int) { ++starts; });
          if (b) prev = seg0 + 32 * w + 31 - __clz(int(b));
        }
        int found;
        int idx = n_win + block_excl_sum<NT>(starts, red, &found);
        n_win += found;
        if (n_win <= kStageMaxTiles && starts > 0) {
          prev = before;
          for (int w = lo; w < hi; ++w) {
            const uint32_t b = bm[w];
            window_starts(b, seg0 + 32 * w, prev, gap, [&](int p, int pv) {
              win_start[idx] = p;
              win_prev[idx] = pv;
              ++idx;
            });
            if (b) prev = seg0 + 32 * w + 31 - __clz(int(b));
          }
        }
        if (last_seg >= 0) prev_seg = last_seg;
        __syncthreads();                            // the bitmap and the windows so far
      }
      if (n_win > kStageMaxTiles) {
        code = kNoTiles;
      } else {
        // tiles per window: window i spans [start_i, end_i], end_i being the
        // set bit before the next window's start (the last set bit for the
        // last window)
        if (tid < 64) {
          int wt = 0, ws = 0, we = 0;
          if (tid < n_win) {
            ws = win_start[tid];
            we = tid + 1 < n_win ? win_prev[tid + 1] : prev_seg;
            wt = (we - ws + 64) / 64;
          }
          const int tincl = wave_inclusive_scan(wt);
          const int total = __shfl(tincl, 63, 64);
          if (tid == 0) tiles_all = total;
          if (FILL && total <= kStageMaxTiles) {
            const int first_tile = tincl - wt;
            const int tp = tile_ptr[g];
            if (tile_ptr[g + 1] - tp != total || tp < 0 || tp + total > n_stage_tiles) {
              if (tid == 0) box[kBoxMismatch] = 1;
            } else if (tid < n_win) {
              for (int m = 0; m < wt; ++m) {
                const int t0 = ws + 64 * m;
                tile_start[tp + first_tile + m] = mn + t0;
                tile_len[tp + first_tile + m] = we - t0 + 1 < 64 ? we - t0 + 1 : 64;
              }
            }
            if (tid < n_win) win_base[tid] = 64 * first_tile - ws;
          }
        }
        __syncthreads();
        n_tiles = tiles_all;
        if (n_tiles > kStageMaxTiles) code = kNoTiles;
      }
    }
  }
  if constexpr (!FILL) {
    if (tid == 0) tile_ptr[g + 1] = code ? code : n_tiles;
    return;
  }
  if (code) {
    if (tid == 0) box[kBoxUnstageable] = 1;
    return;
  }
  // every slot's position in the staged tiles: the last window starting at or
  // before its column, by a binary search (n_win <= 64) where it is not the
  // window of the slot before it
  uint16_t* out = local + gi.offset;
  for (int64_t base = 0; base < slots; base += kRound) {
    if (!held) load(base);
#pragma unroll
    for (int k = 0; k < kVecs; ++k) {
      const int64_t s = base + 4 * int64_t(tid + k * NT);
      if (s >= slots) break;
      int from = 1, to = 0, at = 0;                 // the window's columns and position base
      v4u16 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = c[k][e] - mn;
        if (c[k][e] >= 0 && (r < from || r >= to)) {
          int w = 0;
          for (int step = n_win > 1 ? 1 << (31 - __clz(n_win - 1)) : 0; step > 0; step >>= 1)
            if (w + step < n_win && win_start[w + step] <= r) w += step;
          from = win_start[w];
          to = w + 1 < n_win ? win_start[w + 1] : INT_MAX;
          at = win_base[w];
        }
        v[e] = c[k][e] >= 0 ? uint16_t(at + r) : kStagePad;
      }
      if (vec) {
        __builtin_nontemporal_store(v, reinterpret_cast<v4u16*>(out + s));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (s + e < slots) out[s + e] = v[e];
      }
    }
  }
}

// tile_ptr[1..G] holds per-group counts or codes; turns tile_ptr into the
// exclusive scan (tile_ptr[0] = 0) and writes the total, the largest count
// and which codes there were to the result slot.  One workgroup, eight
// counts a thread and round: the rounds, one chain of load and scan each,
// are what it costs (7813 groups are one round).
constexpr int kScanPer = 8;
__global__ __launch_bounds__(1024) void stage_scan_kernel(int32_t* __restrict__ tile_ptr,
                                                        int32_t n_groups,
                                                        int64_t* __restrict__ box) {
  __shared__ int red[16];
  int carry = 0, biggest = 0, codes = 0;
  for (int32_t base = 0; base < n_groups; base += 1024 * kScanPer) {
    const int32_t i0 = base + int32_t(threadIdx.x) * kScanPer;
    int v[kScanPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) v[k] = i0 + k < n_groups ? tile_ptr[i0 + k + 1] : 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (v[k] < 0) {
        codes |= v[k] == kNoSpan ? 1 : 2;
        v[k] = 0;
      }
      biggest = v[k] > biggest ? v[k] : biggest;
      sum += v[k];
    }
    int all;
    int run = carry + block_excl_sum<1024>(sum, red, &all);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      run += v[k];
      if (i0 + k < n_groups) tile_ptr[i0 + k + 1] = run;
    }
    carry += all;
  }
  biggest = block_max<1024>(biggest, red);
  const int no_span = block_max<1024>(codes & 1, red);
  const int no_tiles = block_max<1024>(codes & 2, red);
  if (threadIdx.x == 0) {
    tile_ptr[0] = 0;
    box[kBoxTotal] = carry;
    box[kBoxMaxTiles] = biggest;
    box[kBoxUnstageable] = no_span | no_tiles;
  }
}

template <bool FILL, int NT>
void launch_waves(const argcsr_matrix* A, int32_t gap, int32_t* tile_ptr, int64_t* box,
                  hipStream_t s) {
  stage_kernel<FILL, NT><<<A->n_groups, NT, 0, s>>>(
      A->groups, A->n_groups, A->block_dim, A->columns, gap, tile_ptr, A->n_stage_tiles,
      A->tile_start, A->tile_len, A->local, box);
}

// The smallest workgroup whose registers hold the average group: fewer waves
// read a group again from L2 in each phase, more wait at barriers for little
// work.  argcsr_stage_plan + argcsr_stage, both passes with their waits, with
// 1 / 2 / 4 waves: 27-point stencil, 3424 slots a group 198 / 158 / 154 us,
// 1708 slots 193 / 182 / 231 us; 5-point Laplacian, 640 slots 74 / 86 / 104 us.
template <bool FILL>
void launch_stage(const argcsr_matrix* A, int32_t gap, int32_t* tile_ptr, int64_t* box,
                  hipStream_t s) {
  const int64_t per_wave = int64_t(A->n_groups) * 64 * kHeldSlots;
  if (A->n_slots <= per_wave) launch_waves<FILL, 64>(A, gap, tile_ptr, box, s);
  else if (A->n_slots <= 2 * per_wave) launch_waves<FILL, 128>(A, gap, tile_ptr, box, s);
  else launch_waves<FILL, 256>(A, gap, tile_ptr, box, s);
}

// Waits for the stream whose kernels write `box`.
int wait_for(Mailbox& box, hipStream_t s) {
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess) {
    box.idle();
    return ARGCSR_OK;
  }
  return fail(ARGCSR_EHIP, "staging: %s", hipGetErrorString(e));
}

int check_stage_input(const argcsr_matrix* A) {
  if (!A) return fail(ARGCSR_EINVAL, "matrix is NULL");
  if (A->n_groups < 0 || A->n_slots < 0 || A->block_dim < 1)
    return fail(ARGCSR_EINVAL, "malformed matrix descriptor");
  if (A->n_slots > INT32_MAX) return fail(ARGCSR_EOVERFLOW, "n_slots exceeds INT32_MAX");
  if (A->n_groups > 0 && (!A->groups || !A->columns))
    return fail(ARGCSR_EINVAL, "staging needs the converted groups and columns");
  return ARGCSR_OK;
}

}  // namespace
}  // namespace argcsr

extern "C" int argcsr_stage_plan(const argcsr_matrix* A, int32_t gap, int32_t* tile_ptr,
                                 int32_t* n_tiles, int32_t* max_group_tiles, void* stream) {
  using namespace argcsr;
  clear_error();
  int rc = check_stage_input(A);
  if (rc) return rc;
  if (gap < 0) return fail(ARGCSR_EINVAL, "gap < 0");
  if (!tile_ptr || !n_tiles) return fail(ARGCSR_EINVAL, "NULL argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  *n_tiles = 0;
  if (max_group_tiles) *max_group_tiles = 0;
  if (A->n_groups == 0) {
    const int32_t zero = 0;
    ARGCSR_HIP(hipMemcpyAsync(tile_ptr, &zero, sizeof(zero), hipMemcpyHostToDevice, s));
    ARGCSR_HIP(hipStreamSynchronize(s));
    return ARGCSR_OK;
  }
  Mailbox box;
  rc = box.init(s);
  if (rc) return rc;
  launch_stage<false>(A, gap, tile_ptr, box.device(), s);
  stage_scan_kernel<<<1, 1024, 0, s>>>(tile_ptr, A->n_groups, box.device());
  rc = wait_for(box, s);
  if (rc) return rc;
  if (box.word(kBoxUnstageable) & 1)
    return fail(ARGCSR_EUNSUPPORTED, "a group's columns span more than %d columns", kStageSpanBits);
  if (box.word(kBoxUnstageable) & 2)
    return fail(ARGCSR_EUNSUPPORTED, "a group needs more than %d tiles of x", kStageMaxTiles);
  *n_tiles = int32_t(box.word(kBoxTotal));
  if (max_group_tiles) *max_group_tiles = int32_t(box.word(kBoxMaxTiles));
  return ARGCSR_OK;
}

extern "C" int argcsr_stage(argcsr_matrix* A, void* stream) {
  using namespace argcsr;
  clear_error();
  int rc = check_stage_input(A);
  if (rc) return rc;
  if (A->stage_gap < 0) return fail(ARGCSR_EINVAL, "stage_gap < 0");
  if (A->n_stage_tiles < 0 || A->stage_max_tiles < 0 || A->stage_max_tiles > kStageMaxTiles)
    return fail(ARGCSR_EINVAL, "malformed staging sizes");
  if (A->n_groups == 0) return ARGCSR_OK;
  if (!A->tile_ptr || !A->local || (A->n_stage_tiles > 0 && (!A->tile_start || !A->tile_len)))
    return fail(ARGCSR_EINVAL, "NULL staging buffer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  Mailbox box;
  rc = box.init(s);
  if (rc) return rc;
  launch_stage<true>(A, A->stage_gap, A->tile_ptr, box.device(), s);
  rc = wait_for(box, s);
  if (rc) return rc;
  if (box.word(kBoxUnstageable))
    return fail(ARGCSR_EUNSUPPORTED, "the matrix cannot be staged with gap %d", A->stage_gap);
  if (box.word(kBoxMismatch))
    return fail(ARGCSR_EINVAL, "tile_ptr was not made by argcsr_stage_plan with this gap");
  return ARGCSR_OK;
}
