// Many ARG-CSR matrices in one launch.
//
// Work items are (matrix, group) pairs in matrix and row order, so waves
// working at the same time gather from the same few x vectors.  Heavy groups
// (a long chunk loop, see schedule.hpp) come first, a workgroup each, split
// over its waves.  All other items are cut, when the batch is made, into
// chunks of about equal cost, a workgroup each: the workgroup reads its
// items' group records into LDS and its waves take them one by one from a
// counter there.  Each group is computed by the same deterministic routine
// as argcsr_spmv, so the results do not depend on which wave takes which
// item.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>
#include <vector>

#include "batch.hpp"
#include "common.hpp"
#include "schedule.hpp"
#include "spmv_kernels.hpp"

namespace argcsr {
namespace {

constexpr int kChunkItems = 64;          // items of a chunk, at most
// Cost of an item besides its slots, in slots (the round trips of a short
// group), and cost of a chunk.  Larger chunks leave the CUs unevenly loaded at
// the end, smaller ones are mostly start-up.  Batches of 48 / 256 matrices of
// 10^3 .. 2*10^5 rows in FP32, half with uniform, half with power-law rows,
// MI355X, us at chunk costs 1200, 2400, 3600, 4800, 7200: 179 / 934, 172 / 887,
// 172 / 877, 169 / 858, 180 / 920; with an item cost of 512 instead 182 / 945 to
// 171 / 874.
constexpr int64_t kItemCost = 128;
constexpr int64_t kChunkCost = 4800;

template <int DT, int W, int U>
__device__ __forceinline__ void run_item(const BatchMat& m, const argcsr_group_info& gi,
                                         int32_t* ends) {
  using Vt = Val<DT>;
  spmv_group<DT, W, U>(gi.first_row, gi.size, gi.offset, gi.chunk_size, global_ptr<const int32_t>(m.tm),
                       global_ptr<const int32_t>(m.columns),
                       global_ptr<const typename Vt::storage>(m.values),
                       XGather<typename Vt::acc>(
                           global_ptr<const typename Vt::acc>(m.x), m.n_cols),
                       m.serial != 0, global_ptr<typename Vt::acc>(m.y), ends);
}

template <int DT, int W, int U>
__device__ __forceinline__ void run_heavy(const BatchMat& m, int32_t g, int32_t* ends,
                                          typename Val<DT>::acc* part_mem, int wv) {
  using Vt = Val<DT>;
  using A = typename Vt::acc;
  const argcsr_group_info gi = load_group(global_ptr<const argcsr_group_info>(m.groups) + g);
  spmv_group_split<DT, W, U>(gi.first_row, gi.size, gi.offset, gi.chunk_size, global_ptr<const int32_t>(m.tm),
                             global_ptr<const int32_t>(m.columns),
                             global_ptr<const typename Vt::storage>(m.values),
                             XGather<A>(global_ptr<const A>(m.x), m.n_cols),
                             m.serial != 0, global_ptr<A>(m.y), ends,
                             reinterpret_cast<A(*)[64 * W]>(part_mem), wv);
}

// Bound by the x gathers: the 29.5 M of the 48-matrix batch above run at
// 179 G/s, where gathers and streams alone reach 185 to 225 G/s.  No workgroup
// waits for another and nothing is counted in device memory: with persistent
// workgroups that took their items from counters there, the 5120 waves' last,
// failing atomics on each counter (about 12 ns each, one after another) cost
// more than the gathers of a small batch.  That batch 225 -> 169 us
// (165 with the records and mappings of spmv_kernels.hpp loaded ahead), 256
// matrices 973 -> 858, eight of up to 2*10^4 rows in BF16 44 -> 22.
template <int DT>
__global__ __launch_bounds__(kSpmvWaves * 64) void batch_spmv_kernel(
    const BatchMat* __restrict__ mats, const int2* __restrict__ heavy, int32_t n_heavy,
    const int2* __restrict__ items, const int32_t* __restrict__ chunk_begin) {
  using A = typename Val<DT>::acc;
  __shared__ int32_t ends[kSpmvWaves][256];
  __shared__ A part_mem[(kSpmvWaves - 1) * 256];
  __shared__ argcsr_group_info recs[kChunkItems];
  __shared__ int32_t mat_of[kChunkItems];
  __shared__ int32_t next;
  const int wv = wave_uniform(int(threadIdx.x >> 6));
  const int32_t b = int32_t(blockIdx.x);

  if (b < n_heavy) {                      // a heavy group, the whole workgroup
    const int2 it = heavy[b];
    const BatchMat& m = mats[it.x];
    switch (m.block_dim) {
      case 64: run_heavy<DT, 1, 8>(m, it.y, ends[0], part_mem, wv); break;
      case 128: run_heavy<DT, 2, 4>(m, it.y, ends[0], part_mem, wv); break;
      default: run_heavy<DT, 4, 2>(m, it.y, ends[0], part_mem, wv); break;
    }
    return;
  }

  // a chunk of the other groups.  Neighbouring chunks go to different XCDs: a
  // contiguous eighth of the items per XCD would keep an x in one L2, but the
  // eighths of a mixed batch differ in gathers by a quarter (172 against 169,
  // 878 against 858 us for the batches above)
  const int32_t ch = b - n_heavy;
  const int32_t i0 = chunk_begin[ch];
  const int32_t count = chunk_begin[ch + 1] - i0;
  const int t = int(threadIdx.x);
  if (t < count) {
    const int2 it = items[i0 + t];
    recs[t] = global_ptr<const argcsr_group_info>(mats[it.x].groups)[it.y];
    mat_of[t] = it.x;
  }
  if (t == 0) next = kSpmvWaves;
  __syncthreads();
  for (int32_t k = wv; k < count;) {
    argcsr_group_info gi = recs[k];
    gi.first_row = wave_uniform(gi.first_row);
    gi.size = wave_uniform(gi.size);
    gi.offset = wave_uniform(gi.offset);
    gi.chunk_size = wave_uniform(gi.chunk_size);
    const BatchMat& m = mats[wave_uniform(mat_of[k])];
    switch (m.block_dim) {
      case 64: run_item<DT, 1, 8>(m, gi, ends[wv]); break;
      case 128: run_item<DT, 2, 4>(m, gi, ends[wv]); break;
      default: run_item<DT, 4, 2>(m, gi, ends[wv]); break;
    }
    int32_t taken = 0;
    if (lane_id() == 0) taken = atomicAdd(&next, 1);
    k = wave_uniform(taken);
  }
}

int launch_kernels(argcsr_batch* b, hipStream_t s) {
  const dim3 grid(b->grid), block(kSpmvWaves * 64);
  auto go = [&](auto* kern) {
    kern<<<grid, block, 0, s>>>(b->d_mats, b->d_heavy, b->n_heavy, b->d_items, b->d_chunks);
  };
  switch (b->dtype) {
    case ARGCSR_F64: go(&batch_spmv_kernel<ARGCSR_F64>); break;
    case ARGCSR_F32: go(&batch_spmv_kernel<ARGCSR_F32>); break;
    case ARGCSR_BF16: go(&batch_spmv_kernel<ARGCSR_BF16>); break;
    default: go(&batch_spmv_kernel<ARGCSR_F16>); break;
  }
  ARGCSR_HIP(hipGetLastError());
  return ARGCSR_OK;
}

void free_batch(argcsr_batch* b) {
  if (!b) return;
  if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  if (b->d_mats) (void)hipFree(b->d_mats);
  if (b->d_items) (void)hipFree(b->d_items);
  if (b->d_heavy) (void)hipFree(b->d_heavy);
  if (b->d_chunks) (void)hipFree(b->d_chunks);
  if (b->last) (void)hipEventDestroy(b->last);
  delete b;
}

}  // namespace

// Builds the work lists on the host from the converted group tables.
int build_batch(int32_t n, const argcsr_matrix* mats, const void* const* xs, void* const* ys,
                argcsr_batch* b) {
  b->n_mats = n;
  b->dtype = mats[0].dtype;
  std::vector<BatchMat> hm(n);
  std::vector<int2> items;
  std::vector<int2> heavy;
  std::vector<int64_t> cost;               // of each item
  std::vector<argcsr_group_info> g;
  for (int32_t m = 0; m < n; ++m) {
    const argcsr_matrix& A = mats[m];
    int rc = check_matrix(&A);
    if (rc) return rc;
    if (A.dtype != b->dtype)
      return fail(ARGCSR_EINVAL, "matrix %d has dtype %d, batch dtype is %d", m, A.dtype, b->dtype);
    if (A.n_groups > 0 && (!xs[m] || !ys[m]))
      return fail(ARGCSR_EINVAL, "matrix %d: x or y is NULL", m);
    if (A.n_groups > 0 && !A.columns)
      return fail(ARGCSR_EINVAL, "matrix %d: a batch reads columns (staging is not used)", m);
    hm[m] = BatchMat{A.groups, A.threads_mapping, A.columns, A.values, xs[m], ys[m],
                     A.block_dim, A.n_groups, A.n_cols,
                     serial_gathers(A.dtype == ARGCSR_F64 ? 8 : A.dtype == ARGCSR_F32 ? 4 : 2,
                                    A.block_dim, A.n_slots, A.n_groups) ? 1 : 0};
    g.resize(size_t(A.n_groups));
    if (A.n_groups > 0)
      ARGCSR_HIP(hipMemcpy(g.data(), A.groups, sizeof(argcsr_group_info) * g.size(),
                           hipMemcpyDeviceToHost));
    const int32_t hc = heavy_chunk_for(A.block_dim, A.n_slots, A.n_groups);
    for (int32_t k = 0; k < A.n_groups; ++k) {
      if (g[k].chunk_size > hc) {
        heavy.push_back(int2{m, k});
      } else {
        items.push_back(int2{m, k});
        cost.push_back(int64_t(g[k].chunk_size) * A.block_dim + kItemCost);
      }
    }
  }
  // matrix-major, row order: waves working at the same time gather from the
  // same few x vectors (sorting by length across matrices measured 13% slower)
  b->n_items = int32_t(items.size());
  b->n_heavy = int32_t(heavy.size());

  ARGCSR_HIP(hipMalloc(&b->d_mats, sizeof(BatchMat) * size_t(std::max(n, 1))));
  ARGCSR_HIP(hipMalloc(&b->d_items, sizeof(int2) * std::max<size_t>(items.size(), 1)));
  ARGCSR_HIP(hipMalloc(&b->d_heavy, sizeof(int2) * std::max<size_t>(heavy.size(), 1)));
  ARGCSR_HIP(hipMemcpy(b->d_mats, hm.data(), sizeof(BatchMat) * size_t(n), hipMemcpyHostToDevice));
  if (!items.empty())
    ARGCSR_HIP(hipMemcpy(b->d_items, items.data(), sizeof(int2) * items.size(),
                         hipMemcpyHostToDevice));
  if (!heavy.empty())
    ARGCSR_HIP(hipMemcpy(b->d_heavy, heavy.data(), sizeof(int2) * heavy.size(),
                         hipMemcpyHostToDevice));
  std::vector<int32_t> chunks{0};
  if (items.empty()) chunks.push_back(0);      // one empty chunk: a launch has a workgroup
  int64_t in_chunk = 0;
  for (size_t i = 0; i < items.size(); ++i) {
    in_chunk += cost[i];
    if (in_chunk >= kChunkCost || int32_t(i) + 1 - chunks.back() == kChunkItems ||
        i + 1 == items.size()) {
      chunks.push_back(int32_t(i) + 1);
      in_chunk = 0;
    }
  }
  ARGCSR_HIP(hipMalloc(&b->d_chunks, sizeof(int32_t) * chunks.size()));
  ARGCSR_HIP(hipMemcpy(b->d_chunks, chunks.data(), sizeof(int32_t) * chunks.size(),
                       hipMemcpyHostToDevice));
  b->grid = b->n_heavy + int32_t(chunks.size()) - 1;
  return ARGCSR_OK;
}

}  // namespace argcsr

extern "C" int argcsr_batch_create(int32_t n_mats, const argcsr_matrix* mats,
                                   const void* const* xs, void* const* ys,
                                   argcsr_batch** out) {
  using namespace argcsr;
  clear_error();
  if (!out) return fail(ARGCSR_EINVAL, "out is NULL");
  *out = nullptr;
  if (n_mats < 1 || !mats || !xs || !ys) return fail(ARGCSR_EINVAL, "empty or NULL batch");
  auto* b = new (std::nothrow) argcsr_batch();
  if (!b) return fail(ARGCSR_ENOMEM, "host allocation failed");
  int rc = build_batch(n_mats, mats, xs, ys, b);
  if (rc) { free_batch(b); return rc; }
  if (hipEventCreateWithFlags(&b->last, hipEventDisableTiming) != hipSuccess) {
    b->last = nullptr;
    free_batch(b);
    return fail(ARGCSR_EHIP, "hipEventCreate failed");
  }
  // capture the kernel into a graph on a private stream
  hipStream_t cs = nullptr;
  if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) {
    free_batch(b);
    return fail(ARGCSR_EHIP, "hipStreamCreate failed");
  }
  hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    rc = launch_kernels(b, cs);
    hipGraph_t graph = nullptr;
    const hipError_t e2 = hipStreamEndCapture(cs, &graph);
    b->graph = graph;
    if (rc == ARGCSR_OK && e2 == hipSuccess)
      e = hipGraphInstantiate(&b->graph_exec, graph, nullptr, nullptr, 0);
    else
      e = e2 != hipSuccess ? e2 : hipErrorUnknown;
  }
  (void)hipStreamDestroy(cs);
  if (e != hipSuccess || rc != ARGCSR_OK) {
    free_batch(b);
    return rc ? rc : fail(ARGCSR_EHIP, "graph capture failed: %s", hipGetErrorString(e));
  }
  *out = b;
  return ARGCSR_OK;
}

extern "C" int argcsr_batch_launch(argcsr_batch* b, void* stream) {
  using namespace argcsr;
  clear_error();
  if (!b) return fail(ARGCSR_EINVAL, "batch is NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rc = launch_kernels(b, s);
  if (rc) return rc;
  ARGCSR_HIP(hipEventRecord(b->last, s));
  b->launched = true;
  return ARGCSR_OK;
}

extern "C" int argcsr_batch_graph_launch(argcsr_batch* b, void* stream) {
  using namespace argcsr;
  clear_error();
  if (!b || !b->graph_exec) return fail(ARGCSR_EINVAL, "batch is NULL or has no graph");
  hipStream_t s = static_cast<hipStream_t>(stream);
  ARGCSR_HIP(hipGraphLaunch(b->graph_exec, s));
  ARGCSR_HIP(hipEventRecord(b->last, s));
  b->launched = true;
  return ARGCSR_OK;
}

extern "C" int argcsr_batch_info(const argcsr_batch* b, int32_t* n_items, int32_t* n_heavy,
                                 int32_t* grid) {
  using namespace argcsr;
  clear_error();
  if (!b) return fail(ARGCSR_EINVAL, "batch is NULL");
  if (n_items) *n_items = b->n_items;
  if (n_heavy) *n_heavy = b->n_heavy;
  if (grid) *grid = b->grid;
  return ARGCSR_OK;
}

extern "C" int argcsr_batch_destroy(argcsr_batch* b) {
  using namespace argcsr;
  clear_error();
  if (b) {
    // the last launch may still be in flight on a caller stream: wait for it
    // alone (launches are ordered on their streams; a caller that launches
    // on several streams at once orders them itself)
    const hipError_t e = b->launched ? hipEventSynchronize(b->last) : hipSuccess;
    free_batch(b);
    if (e != hipSuccess)
      return fail(ARGCSR_EHIP, "waiting for the batch's last launch failed: %s",
                  hipGetErrorString(e));
  }
  return ARGCSR_OK;
}
