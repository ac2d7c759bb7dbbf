// y_m = A_m x_m for a set of matrices in ONE launch, driven by per-matrix
// prefix tables instead of a per-group work list: the first total_heavy
// workgroups take heavy item h = heavy_groups_m[h - heavy_begin[m]] each,
// and then wave i of the rest takes group i - group_begin[m] of the matrix m
// with group_begin[m] <= i < group_begin[m+1].  Used by the serving loop,
// whose set of matrices changes from step to step: the grid is sized on the
// host for each step, so no wave takes work from a shared counter.
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"
#include "schedule.hpp"
#include "spmv_kernels.hpp"

namespace argcsr {

constexpr int kMaxLaunchMats = 512;   // matrices per multi-matrix launch

struct MatWork {
  const argcsr_group_info* groups;
  const int32_t* tm;
  const int32_t* columns;
  const void* values;
  const int32_t* heavy;               // heavy group indices (may be NULL if n_heavy == 0)
  const void* x;
  void* y;
  int32_t block_dim;
  int32_t n_cols;
  int32_t serial;                     // gather mode (serial_gathers)
  int32_t heavy_chunk;                // groups with chunk_size above are in `heavy`
  int32_t group_begin;                // prefix over the launch's matrices
  int32_t heavy_begin;
};

// The largest m in [0, n) with begin of m <= i (the first begin is 0, they do
// not decrease), by the whole wave: lane m looks at matrix m, 64 at a time.
// One round trip; a copy of the prefix in LDS, searched there, cost a
// barrier and a chain of LDS reads more per wave.
__device__ __forceinline__ int32_t find_owner(const MatWork* __restrict__ mw,
                                              int32_t MatWork::* begin, int32_t n, int32_t i) {
  int32_t owner = 0;
  for (int32_t m0 = 0; m0 < n; m0 += 64) {
    const int32_t m = m0 + lane_id();
    const uint64_t at_or_before = __ballot(m < n && mw[m < n ? m : 0].*begin <= i);
    if (at_or_before == 0) break;
    owner = m0 + 63 - __clzll((long long)at_or_before);
  }
  return owner;
}

// All matrices of a launch share T = 64*W (the server converts with one
// block size), so each kernel instance holds one group routine only.
template <int DT, int W, int U>
__global__ __launch_bounds__(kSpmvWaves * 64) void mspmv_kernel(
    const MatWork* __restrict__ mw, int32_t n_mats, int32_t total_groups, int32_t total_heavy) {
  using Vt = Val<DT>;
  using S = typename Vt::storage;
  using A = typename Vt::acc;
  __shared__ int32_t ends[kSpmvWaves][64 * W];
  __shared__ A part_mem[kSpmvWaves - 1][64 * W];
  const int wv = wave_uniform(int(threadIdx.x >> 6));
  const int32_t b = int32_t(blockIdx.x);

  if (b < total_heavy) {                            // a heavy group, the whole workgroup
    const int32_t m = find_owner(mw, &MatWork::heavy_begin, n_mats, b);
    const MatWork& w = mw[m];
    const int32_t g = global_ptr<const int32_t>(w.heavy)[b - w.heavy_begin];
    const argcsr_group_info gi = load_group(global_ptr<const argcsr_group_info>(w.groups) + g);
    spmv_group_split<DT, W, U, false>(
        gi.first_row, gi.size, gi.offset, gi.chunk_size, global_ptr<const int32_t>(w.tm),
        global_ptr<const int32_t>(w.columns), global_ptr<const S>(w.values),
        XGather<A>(global_ptr<const A>(w.x), w.n_cols), w.serial != 0, global_ptr<A>(w.y), ends[0],
        part_mem, wv);
    return;
  }
  // the other groups, one wave each, every XCD a contiguous range of them
  const uint32_t nb = gridDim.x - uint32_t(total_heavy);
  const int32_t i = int32_t(xcd_remap(uint32_t(b - total_heavy), nb)) * kSpmvWaves + wv;
  if (i >= total_groups) return;
  const int32_t m = find_owner(mw, &MatWork::group_begin, n_mats, i);
  const MatWork& w = mw[m];
  const argcsr_group_info gi =
      load_group(global_ptr<const argcsr_group_info>(w.groups) + (i - w.group_begin));
  if (gi.chunk_size > w.heavy_chunk) return;        // done by a heavy workgroup
  spmv_group<DT, W, U, false>(
      gi.first_row, gi.size, gi.offset, gi.chunk_size, global_ptr<const int32_t>(w.tm),
      global_ptr<const int32_t>(w.columns), global_ptr<const S>(w.values),
      XGather<A>(global_ptr<const A>(w.x), w.n_cols), w.serial != 0, global_ptr<A>(w.y), ends[wv]);
}

}  // namespace argcsr
