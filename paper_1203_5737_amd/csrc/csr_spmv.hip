// Plain CSR y = A x on the same GPU: the baseline the ARG-CSR kernel is
// measured against (CSR definition, Sec. 2).  "CSR-vector": V consecutive
// lanes (V a power of two, 1..64) share a row, stride through its nonzeros
// (coalesced), and combine their partial sums with a butterfly over the V
// lanes.  V defaults to the power of two nearest above the mean row length.
//
// Binned variant (still plain CSR, no other storage): the rows are grouped
// by length once (argcsr_csr_bin_rows: bin k < 7 holds the rows of at most
// 2^k nonzeros and more than 2^(k-1), bin 7 the longer ones), and one launch
// gives each bin its own width: 2^k lanes per row, and for bin 7 a 256-lane
// workgroup per row.  A row of bin k < 7 is summed exactly as by the uniform
// kernel with V = 2^k.
#include <hip/hip_runtime.h>

#include <vector>

#include "common.hpp"
#include "scratch.hpp"
#include "values.hpp"

namespace argcsr {
namespace {

constexpr int kCsrBlock = 256;
constexpr int kLongBatch = 8;     // elements of a row of bin 7 a lane loads at a time, or half

// How the rows of bin 7 are read: those of up to `single` elements one element
// a lane after the other, longer ones in batches.  A batch hides the chain of
// column, x and sum, but many workgroups' batches queue their gathers in front
// of each other's loads.  With `streamed` the elements pass by L2 and the
// Infinity Cache.  us, three matrices in turn, FP32 but where marked:
// * Up to kCachedBytes a matrix the Infinity Cache holds the elements from one
//   product to the next: ordinary loads.  Where bin 7 holds nearly all of the
//   matrix only rows over 4096 take batches: over 4096 / all / all streamed, 1000
//   rows of 3000 11.8 / 15.1 / 17.7, 4000 of 1000 20.4 / 21.3 / 26.  Beside other
//   rows, those over 1024, whose round trips the launch takes: over 4096 / over
//   1024 / over 1024 streamed, power-law rows of 10^5 10.0 / 9.3 / 11.3, 3.3*10^5
//   23.2 / 21.9 / 27.6, FP64 30 / 27.3 / 32.3, 10^6 54 / 54 / 59.1 (without
//   batches 61).  With nothing in the caches: 16.9 / 14.5 / 14.7, 33.7 / 31.9 /
//   32.6, FP64 41 / 37 / 34, 75.3 / 75.3 / 70.9, and 1000 rows of 3000, over 4096 /
//   all streamed, 23.6 / 21.0: streamed loads would be the faster there.
// * Beyond, they come from HBM and are streamed.  A lane's first element needs
//   no batch, rows of 1024 just half a one: 70^3 rows of 125, singly / batches of
//   8, 323 / 370, BF16 318 / 407; 10^5 rows of 1000, batches of 4 / 8, 535 / 611,
//   FP64 589 / 659; 3*10^5 rows of 300, batches of 4 / singly, 533 / 582, FP64
//   617 / 627, BF16 588 / 568.  Ordinary loads: 4000 rows of 400 beside 3*10^5 of
//   27 93 against 79, but 96 MB of rows of 3000 63 against 74.
// * Earlier where x does not fit the L2 beside them: power-law rows, streamed /
//   not, FP64 8.5*10^5 (68 MB) 63.4 / 63.0, 10^6 (80 MB) 81.2 / 83.2, FP32
//   1.5*10^6 (80 MB) 94 / 97.
struct LongRows {
  int32_t single;
  bool streamed;
};
constexpr int64_t kCachedBytes = 100 * 1000 * 1000;
constexpr int64_t kCachedBesideX = 75 * 1000 * 1000;
constexpr int64_t kL2Bytes = int64_t(4) << 20;    // of an XCD
constexpr LongRows long_rows(int64_t nnz, int64_t long_nnz, int32_t value_bytes, int32_t n_cols,
                             int32_t x_bytes) {
  const int64_t bytes = nnz * (int64_t(sizeof(int32_t)) + value_bytes);
  const bool x_in_l2 = int64_t(n_cols) * x_bytes <= kL2Bytes;
  if (bytes < (x_in_l2 ? kCachedBytes : kCachedBesideX)) return LongRows{long_nnz >= nnz - nnz / 8 ? 4096 : 1024, false};
  return LongRows{value_bytes == 2 ? 512 : 256, true};
}
constexpr int kBins = ARGCSR_CSR_BINS;      // 8: widths 1, 2, 4, ..., 64, then a workgroup

template <bool STREAMED, typename T>
__device__ __forceinline__ T load_element(const T* p) {
  if constexpr (STREAMED) return __builtin_nontemporal_load(p);
  else return *p;
}

// sum plus fma(val, x[col], ...) over elements k, k + stride, ... below end, in that
// order, U of them loaded at a time: a long row is not one chain of column,
// x and sum after the other.
template <int DT, int U, bool STREAMED = false>
__device__ __forceinline__ typename Val<DT>::acc strided_sum(
    int32_t k, int32_t end, int32_t stride, const int32_t* __restrict__ col,
    const typename Val<DT>::storage* __restrict__ val,
    const typename Val<DT>::acc* __restrict__ x, typename Val<DT>::acc sum = 0) {
  using Vt = Val<DT>;
  using A = typename Vt::acc;
  for (; end - k > (U - 1) * stride; k += U * stride) {
    int32_t c[U];
    typename Vt::storage v[U];
    A xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = load_element<STREAMED>(col + k + u * stride);
      v[u] = load_element<STREAMED>(val + k + u * stride);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) sum = __builtin_fma(Vt::load(v[u]), xv[u], sum);
  }
  for (; k < end; k += stride)
    sum = __builtin_fma(Vt::load(load_element<STREAMED>(val + k)),
                        x[load_element<STREAMED>(col + k)], sum);
  return sum;
}

// As strided_sum over elements k0 + lane, + kCsrBlock, ... below end (k0 the same
// for the wave), the elements left over from whole batches in one batch too:
// one by one, their chains of column and x were half of a row of 10^4.  Lanes
// past the end load the row's last element and do not use it.
template <int DT, int U, bool STREAMED>
__device__ __forceinline__ typename Val<DT>::acc long_row_sum(
    int32_t k0, int32_t end, const int32_t* __restrict__ col,
    const typename Val<DT>::storage* __restrict__ val,
    const typename Val<DT>::acc* __restrict__ x) {
  using Vt = Val<DT>;
  using A = typename Vt::acc;
  const int lane = lane_id();
  A sum = A(0);
  int32_t c[U];
  typename Vt::storage v[U];
  A xv[U];
  for (; end - k0 > (U - 1) * kCsrBlock + 63; k0 += U * kCsrBlock) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = load_element<STREAMED>(col + k0 + lane + u * kCsrBlock);
      v[u] = load_element<STREAMED>(val + k0 + lane + u * kCsrBlock);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) sum = __builtin_fma(Vt::load(v[u]), xv[u], sum);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    c[u] = 0;
    v[u] = 0;
    if (end - k0 > u * kCsrBlock) {
      const int32_t k = min(k0 + lane + u * kCsrBlock, end - 1);
      c[u] = load_element<STREAMED>(col + k);
      v[u] = load_element<STREAMED>(val + k);
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    xv[u] = A(0);
    if (end - k0 > u * kCsrBlock) xv[u] = x[c[u]];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const A t = __builtin_fma(Vt::load(v[u]), xv[u], sum);
    sum = end - k0 > u * kCsrBlock + lane ? t : sum;
  }
  return sum;
}

// Sum of row `row` by V consecutive lanes; lane `sub` of the row strides
// through its nonzeros, then a butterfly over the V lanes.
template <int DT, int V>
__device__ __forceinline__ typename Val<DT>::acc csr_row_sum(
    int64_t row, bool valid, int sub, const int32_t* __restrict__ rp,
    const int32_t* __restrict__ col, const typename Val<DT>::storage* __restrict__ val,
    const typename Val<DT>::acc* __restrict__ x) {
  using A = typename Val<DT>::acc;
  A sum = A(0);
  if (valid) sum = strided_sum<DT, 4>(rp[row] + sub, rp[row + 1], V, col, val, x);
#pragma unroll
  for (int d = V / 2; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
  return sum;
}

template <int DT, int V>
__global__ __launch_bounds__(kCsrBlock) void csr_vector_kernel(
    int32_t n_rows, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
    const typename Val<DT>::storage* __restrict__ val,
    const typename Val<DT>::acc* __restrict__ x, typename Val<DT>::acc* __restrict__ y) {
  constexpr int kRowsPerBlock = kCsrBlock / V;
  const int sub = threadIdx.x % V;
  const int64_t row = int64_t(xcd_remap(blockIdx.x, gridDim.x)) * kRowsPerBlock + threadIdx.x / V;
  const bool valid = row < n_rows;     // all V lanes of a row agree
  const auto sum = csr_row_sum<DT, V>(row, valid, sub, rp, col, val, x);
  if (valid && sub == 0) y[row] = sum;
}

// bin of a row of length L: the smallest k with L <= 2^k, 7 above 64
__host__ __device__ __forceinline__ int row_bin(int32_t L) {
  int k = 0;
  while (k < kBins - 1 && L > (1 << k)) ++k;
  return k;
}

// Workgroups of a binned launch.  Bin 7's come first (its rows take longest).
// Those of the other bins are dealt out in `regions`: region g holds the g-th
// of `regions` equal shares of every bin's rows -- rows ascend within a bin, so
// these lie close together in the matrix -- and each XCD takes an eighth of the
// regions, one after another.  Then the cache lines that hold rows of several
// bins are read by one XCD, while they are in its L2, and not once per bin
// (power-law rows of 10^6, FP64: 105 us with the bins one after another, 90
// so).  Any bins that cover the rows give the
// right result; only the speed depends on how they lie.
struct BinLaunch {
  int32_t row_start[kBins + 1];     // bin k's rows: rows[row_start[k] .. row_start[k+1])
  int32_t blocks[kBins];            // workgroups of bin k
  int32_t per[kBins - 1];           // at most, in one region
  int32_t per_region;               // sum of per
  int32_t log2_regions;             // a power of two, at least the XCD count
  int32_t long_blocks;              // bin 7's, rounded up to a multiple of the XCD count
};
constexpr int kXcds = 8, kLog2Xcds = 3;
constexpr int kRegionBlocks = 64;   // workgroups of a region, about

// Workgroup b of bin k: each team of V lanes sums R rows, their loads in
// flight together.
template <int DT, int V, int R>
__device__ __forceinline__ void binned_rows(const BinLaunch& bl, int k, int32_t b,
                                            const int32_t* __restrict__ rows,
                                            const int32_t* __restrict__ rp,
                                            const int32_t* __restrict__ col,
                                            const typename Val<DT>::storage* __restrict__ val,
                                            const typename Val<DT>::acc* __restrict__ x,
                                            typename Val<DT>::acc* __restrict__ y) {
  using Vt = Val<DT>;
  using A = typename Vt::acc;
  constexpr int kTeams = kCsrBlock / V;
  const int sub = threadIdx.x % V;
  const int32_t* list = rows + bl.row_start[k];
  const int32_t n = bl.row_start[k + 1] - bl.row_start[k];
  const int64_t i0 = int64_t(b) * (kTeams * R) + threadIdx.x / V;
  int32_t row[R], at[R], end[R], c[R];
  typename Vt::storage v[R];
  A xv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) row[r] = i0 + r * kTeams < n ? list[i0 + r * kTeams] : -1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    at[r] = row[r] >= 0 ? rp[row[r]] + sub : 0;
    end[r] = row[r] >= 0 ? rp[row[r] + 1] : 0;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool has = at[r] < end[r];
    c[r] = has ? col[at[r]] : -1;
    v[r] = has ? val[at[r]] : typename Vt::storage(0);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) xv[r] = c[r] >= 0 ? x[c[r]] : A(0);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    A sum = A(0);
    if (c[r] >= 0) sum = __builtin_fma(Vt::load(v[r]), xv[r], sum);
    // rows of bin k have at most V nonzeros; bins made for another matrix
    // may hold longer ones
    if (end[r] - at[r] > V) sum = strided_sum<DT, 1>(at[r] + V, end[r], V, col, val, x, sum);
#pragma unroll
    for (int d = V / 2; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (row[r] >= 0 && sub == 0) y[row[r]] = sum;
  }
}

// Bound by the x gathers on power-law rows and by the CSR stream on regular
// ones.  MI355X: power-law rows of 10^6 FP64 125 us -> 81 (long rows first and
// loaded eight elements at a time a lane, regions, a workgroup per long row),
// 27-point stencil 100^3 FP64 171 -> 105.  The code for bin 7 sets the
// registers of every workgroup: with batches of 16 the other bins kept 5 waves
// a SIMD of 8 (that stencil 138 us, in BF16 176 against 124).
template <int DT, int R, bool STREAMED>
__global__ __launch_bounds__(kCsrBlock) void csr_binned_kernel(
    BinLaunch bl, const int32_t* __restrict__ rows, const int32_t* __restrict__ rp,
    const int32_t* __restrict__ col, const typename Val<DT>::storage* __restrict__ val,
    const typename Val<DT>::acc* __restrict__ x, typename Val<DT>::acc* __restrict__ y,
    int32_t single) {
  using A = typename Val<DT>::acc;
  constexpr int kBlockWaves = kCsrBlock / 64;
  int k = kBins - 1;
  int32_t b = int32_t(blockIdx.x);
  if (b >= bl.long_blocks) {
    b -= bl.long_blocks;
    const uint32_t q = uint32_t(b) / kXcds;      // of this XCD's workgroups
    const uint32_t mine = q / uint32_t(bl.per_region);
    const uint32_t region = uint32_t(b % kXcds) * (1u << (bl.log2_regions - kLog2Xcds)) + mine;
    int32_t j = int32_t(q - mine * uint32_t(bl.per_region));
    for (k = kBins - 2; k > 0 && j >= bl.per[k]; --k) j -= bl.per[k];
    const int32_t first = int32_t(uint64_t(uint32_t(bl.blocks[k])) * region >> bl.log2_regions);
    const int32_t last = int32_t(uint64_t(uint32_t(bl.blocks[k])) * (region + 1) >> bl.log2_regions);
    b = first + j;
    if (b >= last) return;
  } else if (b >= bl.blocks[k]) {
    return;
  }
  switch (k) {
    case 0: binned_rows<DT, 1, R>(bl, k, b, rows, rp, col, val, x, y); return;
    case 1: binned_rows<DT, 2, R>(bl, k, b, rows, rp, col, val, x, y); return;
    case 2: binned_rows<DT, 4, R>(bl, k, b, rows, rp, col, val, x, y); return;
    case 3: binned_rows<DT, 8, R>(bl, k, b, rows, rp, col, val, x, y); return;
    case 4: binned_rows<DT, 16, R>(bl, k, b, rows, rp, col, val, x, y); return;
    case 5: binned_rows<DT, 32, R>(bl, k, b, rows, rp, col, val, x, y); return;
    case 6: binned_rows<DT, 64, R>(bl, k, b, rows, rp, col, val, x, y); return;
    default: break;
  }
  // bin 7: a row by the workgroup's 256 lanes, wave sums added in wave order.
  // (Four rows a workgroup, a wave each up to 1024 nonzeros, took a third longer
  // on power-law rows of 4*10^4 to 4*10^5.)  A row of 10^4 takes one CU 10 to 20
  // us, at 2.4 to 5 cycles a gather.
  __shared__ A part[kBlockWaves];
  const int wv = wave_uniform(int(threadIdx.x >> 6));
  const int32_t row = rows[bl.row_start[k] + b];
  const int32_t begin = rp[row], end = rp[row + 1];
  const int32_t k0 = begin + wv * 64;
  A sum = end - begin <= single
              ? strided_sum<DT, 1, STREAMED>(k0 + lane_id(), end, kCsrBlock, col, val, x)
          : end - begin <= kLongBatch / 2 * kCsrBlock
              ? long_row_sum<DT, kLongBatch / 2, STREAMED>(k0, end, col, val, x)
              : long_row_sum<DT, kLongBatch, STREAMED>(k0, end, col, val, x);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
  if (lane_id() == 0) part[wv] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    A t = part[0];
#pragma unroll
    for (int w = 1; w < kBlockWaves; ++w) t += part[w];
    y[row] = t;
  }
}

// Binning: per workgroup of 256 rows, the count of each bin (pass 1), and
// the rows written to their bin's range in ascending order (pass 2) at the
// offsets the host computes from the counts.
__global__ __launch_bounds__(kCsrBlock) void bin_count_kernel(int32_t n_rows,
                                                            const int32_t* __restrict__ rp,
                                                            int32_t* __restrict__ counts) {
  __shared__ int32_t c[kBins];
  if (threadIdx.x < kBins) c[threadIdx.x] = 0;
  __syncthreads();
  const int64_t r = int64_t(blockIdx.x) * kCsrBlock + threadIdx.x;
  if (r < n_rows) atomicAdd(&c[row_bin(rp[r + 1] - rp[r])], 1);
  __syncthreads();
  if (threadIdx.x < kBins) counts[int64_t(blockIdx.x) * kBins + threadIdx.x] = c[threadIdx.x];
}

__global__ __launch_bounds__(kCsrBlock) void bin_scatter_kernel(int32_t n_rows,
                                                              const int32_t* __restrict__ rp,
                                                              const int32_t* __restrict__ offsets,
                                                              int32_t* __restrict__ rows) {
  __shared__ int32_t wave_counts[kCsrBlock / 64][kBins];
  const int lane = lane_id(), w = int(threadIdx.x >> 6);
  const int64_t r = int64_t(blockIdx.x) * kCsrBlock + threadIdx.x;
  const int bin = r < n_rows ? row_bin(rp[r + 1] - rp[r]) : -1;
  // rank among this wave's lanes of the same bin, and the wave's counts
  int rank = 0;
#pragma unroll
  for (int k = 0; k < kBins; ++k) {
    const uint64_t m = __ballot(bin == k);
    if (bin == k) rank = __popcll(m & ((uint64_t(1) << lane) - 1));
    if (lane == 0) wave_counts[w][k] = __popcll(m);
  }
  __syncthreads();
  if (bin >= 0) {
    int before = 0;
    for (int q = 0; q < w; ++q) before += wave_counts[q][bin];
    rows[offsets[int64_t(blockIdx.x) * kBins + bin] + before + rank] = int32_t(r);
  }
}

template <int DT, int V>
void launch(int32_t n_rows, const int32_t* rp, const int32_t* col, const void* val,
            const void* x, void* y, hipStream_t s) {
  using Vt = Val<DT>;
  constexpr int kRowsPerBlock = kCsrBlock / V;
  const int blocks = int((int64_t(n_rows) + kRowsPerBlock - 1) / kRowsPerBlock);
  csr_vector_kernel<DT, V><<<blocks, kCsrBlock, 0, s>>>(
      n_rows, rp, col, static_cast<const typename Vt::storage*>(val),
      static_cast<const typename Vt::acc*>(x), static_cast<typename Vt::acc*>(y));
}

template <int DT>
void launch_v(int V, int32_t n_rows, const int32_t* rp, const int32_t* col, const void* val,
              const void* x, void* y, hipStream_t s) {
  switch (V) {
    case 1: launch<DT, 1>(n_rows, rp, col, val, x, y, s); break;
    case 2: launch<DT, 2>(n_rows, rp, col, val, x, y, s); break;
    case 4: launch<DT, 4>(n_rows, rp, col, val, x, y, s); break;
    case 8: launch<DT, 8>(n_rows, rp, col, val, x, y, s); break;
    case 16: launch<DT, 16>(n_rows, rp, col, val, x, y, s); break;
    case 32: launch<DT, 32>(n_rows, rp, col, val, x, y, s); break;
    default: launch<DT, 64>(n_rows, rp, col, val, x, y, s); break;
  }
}

}  // namespace
}  // namespace argcsr

extern "C" int argcsr_csr_spmv(int32_t n_rows, int32_t n_cols, int64_t nnz,
                               const int32_t* row_ptr, const int32_t* col, const void* val,
                               int32_t dtype, int32_t lanes_per_row, const void* x, void* y,
                               void* stream) {
  using namespace argcsr;
  clear_error();
  if (n_rows < 0 || n_cols < 0 || nnz < 0) return fail(ARGCSR_EINVAL, "negative size");
  if (dtype < ARGCSR_F64 || dtype > ARGCSR_F16) return fail(ARGCSR_EINVAL, "unknown dtype %d", dtype);
  if (lanes_per_row != 0 &&
      (lanes_per_row < 1 || lanes_per_row > 64 || (lanes_per_row & (lanes_per_row - 1))))
    return fail(ARGCSR_EINVAL, "lanes_per_row must be 0 or a power of two in [1, 64]");
  if (n_rows == 0) return ARGCSR_OK;
  if (!row_ptr || !x || !y || (nnz > 0 && (!col || !val)))
    return fail(ARGCSR_EINVAL, "NULL device buffer");
  if (x == y) return fail(ARGCSR_EINVAL, "y must not alias x");
  int V = lanes_per_row;
  if (V == 0) {
    const double mean = double(nnz) / double(n_rows);
    V = 1;
    while (V < 64 && V < mean) V <<= 1;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (dtype) {
    case ARGCSR_F64: launch_v<ARGCSR_F64>(V, n_rows, row_ptr, col, val, x, y, s); break;
    case ARGCSR_F32: launch_v<ARGCSR_F32>(V, n_rows, row_ptr, col, val, x, y, s); break;
    case ARGCSR_BF16: launch_v<ARGCSR_BF16>(V, n_rows, row_ptr, col, val, x, y, s); break;
    default: launch_v<ARGCSR_F16>(V, n_rows, row_ptr, col, val, x, y, s); break;
  }
  ARGCSR_HIP(hipGetLastError());
  return ARGCSR_OK;
}

namespace argcsr {
namespace {

// Rows of a team: four where one bin holds at least half of the workgroups
// (at one row a team) -- rows of about one length -- and else one.  Four rows'
// loads in flight hide the chain of list, offsets, element and x: FP64
// 27-point stencil 100^3 171 us before, 190 with one, 134 with two, 105 with
// four; uniform 5..50 nonzeros 56 / 55 / 50 / 49.  But rows of mixed lengths
// share cache lines across bins (see BinLaunch), and four times the rows in
// flight no longer fit the XCD's 4-MB L2: power-law rows of 10^6, FP64, 90 /
// 95 / 101 us with one, two, four.
int team_rows(const int32_t* bin_start) {
  int64_t most = 0, all = 0;
  for (int k = 0; k < kBins - 1; ++k) {
    const int64_t blocks = ((int64_t(bin_start[k + 1]) - bin_start[k]) << k) / kCsrBlock;
    most = blocks > most ? blocks : most;
    all += blocks;
  }
  return 2 * most >= all ? 4 : 1;
}

template <int DT>
void launch_binned(const BinLaunch& bl, int team, int32_t blocks, int64_t nnz, int64_t long_nnz,
                   int32_t n_cols, const int32_t* rows, const int32_t* rp, const int32_t* col, const void* val,
                   const void* x, void* y, hipStream_t s) {
  using Vt = Val<DT>;
  const LongRows lr = long_rows(nnz, long_nnz, int32_t(sizeof(typename Vt::storage)), n_cols,
                                int32_t(sizeof(typename Vt::acc)));
  auto* kern = team == 4 ? lr.streamed ? &csr_binned_kernel<DT, 4, true>
                                       : &csr_binned_kernel<DT, 4, false>
                         : lr.streamed ? &csr_binned_kernel<DT, 1, true>
                                       : &csr_binned_kernel<DT, 1, false>;
  kern<<<blocks, kCsrBlock, 0, s>>>(
      bl, rows, rp, col, static_cast<const typename Vt::storage*>(val),
      static_cast<const typename Vt::acc*>(x), static_cast<typename Vt::acc*>(y), lr.single);
}

}  // namespace
}  // namespace argcsr

extern "C" int argcsr_csr_bin_rows(int32_t n_rows, const int32_t* row_ptr, int32_t* rows,
                                   int32_t* bin_start, void* stream) {
  using namespace argcsr;
  clear_error();
  if (n_rows < 0) return fail(ARGCSR_EINVAL, "n_rows < 0");
  if (!bin_start) return fail(ARGCSR_EINVAL, "bin_start is NULL");
  for (int k = 0; k <= kBins; ++k) bin_start[k] = 0;
  if (n_rows == 0) return ARGCSR_OK;
  if (!row_ptr || !rows) return fail(ARGCSR_EINVAL, "NULL device buffer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t blocks = (int64_t(n_rows) + kCsrBlock - 1) / kCsrBlock;
  const size_t bytes = sizeof(int32_t) * size_t(blocks) * kBins;
  DeviceScratch ws;
  const int rc = ws.alloc(bytes, s);
  if (rc) return rc;
  int32_t* d_counts = static_cast<int32_t*>(ws.ptr());
  bin_count_kernel<<<dim3(uint32_t(blocks)), kCsrBlock, 0, s>>>(n_rows, row_ptr, d_counts);
  std::vector<int32_t> h(size_t(blocks) * kBins);
  hipError_t e = hipMemcpyAsync(h.data(), d_counts, bytes, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(ARGCSR_EHIP, "binning counts: %s", hipGetErrorString(e));
  // offsets: bin by bin, workgroup by workgroup (rows ascend within a bin)
  int64_t total = 0;
  for (int k = 0; k < kBins; ++k) {
    bin_start[k] = int32_t(total);
    for (int64_t b = 0; b < blocks; ++b) {
      const int32_t c = h[size_t(b) * kBins + k];
      h[size_t(b) * kBins + k] = int32_t(total);
      total += c;
    }
  }
  bin_start[kBins] = int32_t(total);
  e = hipMemcpyAsync(d_counts, h.data(), bytes, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    bin_scatter_kernel<<<dim3(uint32_t(blocks)), kCsrBlock, 0, s>>>(n_rows, row_ptr, d_counts,
                                                                   rows);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(ARGCSR_EHIP, "binning: %s", hipGetErrorString(e));
  ws.idle();
  return ARGCSR_OK;
}

extern "C" int argcsr_csr_spmv_binned(int32_t n_rows, int32_t n_cols, int64_t nnz,
                                      const int32_t* row_ptr, const int32_t* col, const void* val,
                                      int32_t dtype, const int32_t* rows,
                                      const int32_t* bin_start, const void* x, void* y,
                                      void* stream) {
  using namespace argcsr;
  clear_error();
  if (n_rows < 0 || n_cols < 0 || nnz < 0) return fail(ARGCSR_EINVAL, "negative size");
  if (dtype < ARGCSR_F64 || dtype > ARGCSR_F16) return fail(ARGCSR_EINVAL, "unknown dtype %d", dtype);
  if (!bin_start) return fail(ARGCSR_EINVAL, "bin_start is NULL");
  if (bin_start[0] != 0 || bin_start[kBins] != n_rows)
    return fail(ARGCSR_EINVAL, "bin_start does not cover the %d rows", n_rows);
  for (int k = 0; k < kBins; ++k)
    if (bin_start[k + 1] < bin_start[k]) return fail(ARGCSR_EINVAL, "bin_start decreases");
  const int team = team_rows(bin_start);
  BinLaunch bl{};
  int64_t blocks = 0;                 // of the bins but the last
  int64_t long_nnz = nnz;             // elements of the last bin, at least
  for (int k = 0; k < kBins; ++k) {
    bl.row_start[k] = bin_start[k];
    const int64_t cnt = bin_start[k + 1] - bin_start[k];
    const int64_t per = k < kBins - 1 ? team * (kCsrBlock >> k) : 1;   // rows per workgroup
    bl.blocks[k] = int32_t((cnt + per - 1) / per);
    if (k < kBins - 1) blocks += bl.blocks[k], long_nnz -= cnt << k;
  }
  bl.row_start[kBins] = bin_start[kBins];
  bl.long_blocks = (bl.blocks[kBins - 1] + kXcds - 1) / kXcds * kXcds;
  bl.log2_regions = kLog2Xcds;
  while ((int64_t(kRegionBlocks) << bl.log2_regions) < blocks) ++bl.log2_regions;
  for (int k = 0; k < kBins - 1; ++k) {
    bl.per[k] = int32_t((int64_t(bl.blocks[k]) + (1 << bl.log2_regions) - 1) >> bl.log2_regions);
    bl.per_region += bl.per[k];
  }
  if (bl.per_region < 1) bl.per_region = 1;      // (no division by 0; nothing to do)
  const int64_t grid = bl.long_blocks + (blocks > 0 ? int64_t(bl.per_region) << bl.log2_regions : 0);
  if (n_rows == 0) return ARGCSR_OK;
  if (!row_ptr || !rows || !x || !y || (nnz > 0 && (!col || !val)))
    return fail(ARGCSR_EINVAL, "NULL device buffer");
  if (x == y) return fail(ARGCSR_EINVAL, "y must not alias x");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int32_t nb = int32_t(grid);
  auto go = [&](auto* launch) {
    launch(bl, team, nb, nnz, long_nnz, n_cols, rows, row_ptr, col, val, x, y, s);
  };
  switch (dtype) {
    case ARGCSR_F64: go(&launch_binned<ARGCSR_F64>); break;
    case ARGCSR_F32: go(&launch_binned<ARGCSR_F32>); break;
    case ARGCSR_BF16: go(&launch_binned<ARGCSR_BF16>); break;
    default: go(&launch_binned<ARGCSR_F16>); break;
  }
  ARGCSR_HIP(hipGetLastError());
  return ARGCSR_OK;
}
