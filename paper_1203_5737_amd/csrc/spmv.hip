// y = A x for an ARG-CSR matrix on gfx950 (Sec. 4 of the paper: chunk
// partial sums, then per-row sums of the partial sums).
//
// Mapping to CDNA4 (a wave has 64 lanes):
//   - one wave per group; with T = 64*W chunks per group, lane i owns chunks
//     i, i+64, ..., i+64*(W-1) ("sub-blocks" w = 0..W-1).  A group's slots
//     for step j are T consecutive values/columns, so every load is a
//     contiguous, fully coalesced wave-wide access (the paper's column-major
//     chunk storage, Sec. 3);
//   - the group struct is read with scalar loads (wave-uniform); no
//     workgroup barrier is needed anywhere;
//   - the threads mapping is turned into a bitmask of row-end chunks (chunk
//     tm[l]-1 ends row l) through a small per-wave LDS table and a ballot;
//   - each chunk sums value*x[column] over its slots, stopping at the first
//     artificial zero (column -1); a wave leaves the loop once every lane
//     has hit padding (Sec. 4);
//   - row sums are a segmented inclusive scan across lanes (segments = rows,
//     delimited by the row-end mask), carried from one sub-block to the next;
//     the lane holding a row's last chunk writes y[first_row + row].
//     Summation order is fixed by the layout, so results are deterministic.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "spmv_kernels.hpp"
#include "spmv_staged.hpp"

namespace argcsr {
namespace {

template <int DT, int W, int U>
void launch(const argcsr_matrix* A, const void* x, void* y, hipStream_t s) {
  using Vt = Val<DT>;
  const bool sched = A->heavy_groups != nullptr && A->n_heavy > 0;
  const int32_t n_heavy = sched ? A->n_heavy : 0;
  const int32_t heavy_chunk = sched ? A->heavy_chunk : INT32_MAX;
  const int blocks = n_heavy + (A->n_groups + kSpmvWaves - 1) / kSpmvWaves;
  constexpr int32_t kBytes = int32_t(sizeof(typename Vt::storage));
  const bool serial = serial_gathers(kBytes, A->block_dim, A->n_slots, A->n_groups);
  const bool wait = wait_for_mapping(kBytes, A->block_dim, A->n_rows, A->n_slots, A->n_groups,
                                     n_heavy);
  auto* kern = wait ? &argcsr_spmv_kernel<DT, W, U, true> : &argcsr_spmv_kernel<DT, W, U, false>;
  kern<<<blocks, kSpmvWaves * 64, 0, s>>>(
      A->groups, A->n_groups, A->threads_mapping, A->columns,
      static_cast<const typename Vt::storage*>(A->values),
      static_cast<const typename Vt::acc*>(x), A->n_cols, static_cast<typename Vt::acc*>(y),
      A->heavy_groups, n_heavy, heavy_chunk, serial ? 1 : 0);
}

template <int DT, int W, int U, bool XLDS>
int launch_staged(const argcsr_matrix* A, const void* x, void* y, hipStream_t s) {
  using Vt = Val<DT>;
  const bool sched = A->heavy_groups != nullptr && A->n_heavy > 0;
  const int32_t n_heavy = sched ? A->n_heavy : 0;
  const int32_t heavy_chunk = sched ? A->heavy_chunk : INT32_MAX;
  const int blocks = n_heavy + (A->n_groups + kSpmvWaves - 1) / kSpmvWaves;
  const int32_t lds_tiles = A->stage_max_tiles > 0 ? A->stage_max_tiles : 1;
  const size_t lds = size_t(kSpmvWaves) * staged_region_bytes<DT, W, XLDS>(lds_tiles);
  auto* kern = &argcsr_spmv_staged_kernel<DT, W, U, XLDS>;
  if (lds > 64 * 1024)
    ARGCSR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
  kern<<<blocks, kSpmvWaves * 64, lds, s>>>(
      A->groups, A->n_groups, A->threads_mapping, A->local,
      static_cast<const typename Vt::storage*>(A->values), A->tile_ptr, A->tile_start,
      A->tile_len, lds_tiles,
      static_cast<const typename Vt::acc*>(x), A->n_cols, static_cast<typename Vt::acc*>(y),
      A->heavy_groups, n_heavy, heavy_chunk);
  return ARGCSR_OK;
}

// Steps per load batch of the staged kernel, chosen by a sweep (MI355X, x in
// LDS): large batches put a small matrix's few waves through fewer round trips
// but cost registers, and a group shorter than a batch goes step by step.  us
// for the 27-point stencil of 128^3 and 70^3 rows and the 5-point one of 900^2,
// the choice first:
//   FP64  W = 1:  8 101 / 20 / 13.3, 16 102 / 21 / 16.5, 4 102 / 22 / 12.2
//         W = 2:  3 97 / 19 / 11.8, 2 97 / 19 / 11.9, 4 98 / 20 / 11.9
//         W = 4:  2 95 / 21 / 13.1, 1 97 / 24 / 12.9
//   BF16  W = 1:  5 52 / 12 / 8.5, 8 52 / 13 / 11.7, 4 55 / 13 / 9.1
//         W = 2:  3 48 / 13 / 8.6, 2 47 / 15 / 8.0, 4 49 / 13 / 8.7
//         W = 4:  2 47 / 17 / 8.9, 3 45 / 15 / 10.7, 4 51 / 17 / 10.2
// FP32 orders them the same.  With x gathered these steps take, where the plain
// kernel's (8 / 4 / 2 for W = 1 / 2 / 4) and waits between the loads of a batch did
// before: FP64 W = 1 121 / 24 / 13.6 (124 / 25 / 13.4), W = 2 118 / 23 / 12.6 (118 /
// 35 / 15.3), W = 4 113 / 28 / 14.2 (120 / 49 / 17.1); BF16 W = 1 56 / 13 / 8.6 (89 /
// 22 / 12.0), W = 2 55 / 14 / 8.7 (56 / 17 / 11.2), W = 4 56 / 21 / 9.7 (55 / 26 / 11.2).
template <int DT, int W>
constexpr int staged_steps() {
  if (sizeof(typename Val<DT>::acc) == 8) return W == 1 ? 8 : W == 2 ? 3 : 2;
  return W == 1 ? 5 : W == 2 ? 3 : 2;
}

template <int DT, int W, int U>
int launch_w(const argcsr_matrix* A, const void* x, void* y, hipStream_t s) {
  if (!A->local) {
    launch<DT, W, U>(A, x, y, s);
    return ARGCSR_OK;
  }
  constexpr int kSteps = staged_steps<DT, W>();
  return A->stage_lds ? launch_staged<DT, W, kSteps, true>(A, x, y, s)
                      : launch_staged<DT, W, kSteps, false>(A, x, y, s);
}

template <int DT>
int launch_dt(const argcsr_matrix* A, const void* x, void* y, hipStream_t s) {
  switch (A->block_dim) {
    case 64: return launch_w<DT, 1, 8>(A, x, y, s);
    case 128: return launch_w<DT, 2, 4>(A, x, y, s);
    default: return launch_w<DT, 4, 2>(A, x, y, s);
  }
}

}  // namespace

int check_matrix(const argcsr_matrix* A) {
  if (!A) return fail(ARGCSR_EINVAL, "matrix is NULL");
  if (A->n_rows < 0 || A->n_cols < 0 || A->n_groups < 0 || A->n_slots < 0)
    return fail(ARGCSR_EINVAL, "negative size in matrix descriptor");
  if (A->block_dim != 64 && A->block_dim != 128 && A->block_dim != 256)
    return fail(ARGCSR_EUNSUPPORTED, "block_dim %d: the GPU kernels take 64, 128 or 256",
                A->block_dim);
  if (A->dtype < ARGCSR_F64 || A->dtype > ARGCSR_F16)
    return fail(ARGCSR_EINVAL, "unknown dtype %d", A->dtype);
  if (A->n_slots > INT32_MAX) return fail(ARGCSR_EOVERFLOW, "n_slots exceeds INT32_MAX");
  if (int64_t(A->n_cols) * (A->dtype == ARGCSR_F64 ? 8 : 4) > kMaxVectorBytes)
    return fail(ARGCSR_EUNSUPPORTED, "x of %d columns exceeds the %lld-byte gather range",
                A->n_cols, (long long)kMaxVectorBytes);
  if (A->n_groups > 0 && (!A->groups || !A->threads_mapping || !A->values ||
                          (!A->columns && !A->local)))
    return fail(ARGCSR_EINVAL, "NULL device buffer in matrix descriptor");
  if (A->local) {
    if (A->n_stage_tiles < 0 || A->stage_max_tiles < 0 || A->stage_max_tiles > kStageMaxTiles)
      return fail(ARGCSR_EINVAL, "malformed staging sizes");
    if (!A->tile_ptr || (A->n_stage_tiles > 0 && (!A->tile_start || !A->tile_len)))
      return fail(ARGCSR_EINVAL, "NULL staging buffer in matrix descriptor");
  }
  if (A->heavy_groups && (A->n_heavy < 0 || A->n_heavy > A->n_groups ||
                          A->heavy_chunk != heavy_chunk_for(A->block_dim, A->n_slots,
                                                            A->n_groups)))
    return fail(ARGCSR_EINVAL, "heavy-group schedule does not match the matrix");
  return ARGCSR_OK;
}

}  // namespace argcsr

extern "C" int argcsr_spmv(const argcsr_matrix* A, const void* x, void* y, void* stream) {
  using namespace argcsr;
  clear_error();
  int rc = check_matrix(A);
  if (rc) return rc;
  if (A->n_groups == 0) return ARGCSR_OK;
  if (!x || !y) return fail(ARGCSR_EINVAL, "x or y is NULL");
  if (x == y) return fail(ARGCSR_EINVAL, "y must not alias x");
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (A->dtype) {
    case ARGCSR_F64: rc = launch_dt<ARGCSR_F64>(A, x, y, s); break;
    case ARGCSR_F32: rc = launch_dt<ARGCSR_F32>(A, x, y, s); break;
    case ARGCSR_BF16: rc = launch_dt<ARGCSR_BF16>(A, x, y, s); break;
    default: rc = launch_dt<ARGCSR_F16>(A, x, y, s); break;
  }
  if (rc) return rc;
  ARGCSR_HIP(hipGetLastError());
  return ARGCSR_OK;
}
