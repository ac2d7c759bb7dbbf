// Launch-schedule constants shared by host planning and the SpMV kernels.
#pragma once

#include <cstdint>

namespace argcsr {

constexpr int kSpmvWaves = 4;   // waves per SpMV workgroup
// x is gathered through 32-bit buffer offsets; a column -1 must land past the end
constexpr int64_t kMaxVectorBytes = 0xFFFFFFF0ll;
constexpr int kLoadSteps = 8;   // chunk steps loaded ahead per lane (U * W)

// A group is "heavy" when one wave would need many more rounds of loads for
// it than the matrix's typical group: at least kHeavyRounds rounds of
// kLoadSteps steps, and more than kHeavyMeanFactor times the mean chunk size.
// Heavy groups are listed at conversion time, dispatched first and processed
// by all waves of a workgroup, each taking a contiguous share of the chunk
// steps; on regular matrices no group is heavy.  Block dims without a GPU
// kernel get no heavy groups.
constexpr int kHeavyRounds = 4;
constexpr int kHeavyMeanFactor = 4;
__host__ __device__ constexpr int32_t heavy_chunk_for(int32_t block_dim, int64_t n_slots,
                                                      int32_t n_groups) {
  const int32_t by_rounds = block_dim == 64 ? kHeavyRounds * kLoadSteps
                          : block_dim == 128 ? kHeavyRounds * kLoadSteps / 2
                          : block_dim == 256 ? kHeavyRounds * kLoadSteps / 4
                          : INT32_MAX;
  if (by_rounds == INT32_MAX || n_groups <= 0) return by_rounds;
  const int64_t mean_chunk = (n_slots + int64_t(n_groups) * block_dim - 1) /
                             (int64_t(n_groups) * block_dim);
  const int64_t by_mean = kHeavyMeanFactor * mean_chunk;
  return by_rounds > by_mean ? by_rounds : int32_t(by_mean < INT32_MAX ? by_mean : INT32_MAX);
}

// Gather mode of the chunk loop: serial (one gather at a time, each FMA
// right after it) for 8-byte values when the mean chunk loop spans at least
// two load batches -- there the value stream is the limit and the paced
// gathers measured faster (27-point stencil, FP64: 140 vs 149 us) -- and
// batched (all gathers of a batch in flight) otherwise (power-law rows,
// FP64: 81 vs 86 us; every FP32 case).
__host__ __device__ constexpr bool serial_gathers(int32_t value_bytes, int32_t block_dim,
                                                  int64_t n_slots, int32_t n_groups) {
  if (value_bytes != 8 || n_groups <= 0 || block_dim <= 0) return false;
  const int64_t steps_per_batch = block_dim >= kLoadSteps * 64 ? 1 : kLoadSteps * 64 / block_dim;
  const int64_t mean_chunk = n_slots / (int64_t(n_groups) * block_dim);
  return mean_chunk >= 2 * steps_per_batch;
}

// When a product's groups of one wave load their threads mapping: in flight
// with the first chunk loads, or waited for before them (true).  Sooner is
// better where the waves of the light groups are many; but they also get
// between the gathers of a heavy group, whose row of some 10^4 a CU takes
// longer for than for its share of a small matrix, and in 4-byte values at T =
// 64 between their own where chunks are long and rows irregular.  us, FP32
// unless marked, waited for / in flight:
//   power-law rows, T = 64, 10^5 11.9 / 13.1, 2*10^5 14.6 / 15.9, 2.7*10^5
//   18.7 / 18.8, 10^6 55.6 / 53.0; T = 128, 8*10^4 11.8 / 12.1, 2*10^5 17.2 /
//   17.6, 2.3*10^5 19.5 / 19.1; T = 256, 6*10^4 12.3 / 13.0, 1.25*10^5 14.7 /
//   14.5; FP16, T = 128, 6*10^4 10.4 / 11.0, 2.7*10^5 19.8 / 19.8; FP64, T = 64,
//   10^5 15.0 / 15.9, 1.5*10^5 17.9 / 17.3, T = 128 10^5 15.5 / 13.6;
//   uniform rows, T = 64, chunks of 1 (5*10^5 rows) 116 / 107, of 5 69 / 75, of 9
//   73 / 83, of 27 92 / 98; T = 128 of 27 98.8 / 97.7; BF16, T = 64, of 27 93.7 / 93.1;
//   full groups, T = 64: 5-point Laplacian of 10^6 11.1 / 10.4, 27-point stencil 40.1
//   / 40.0.
// Power-law rows have 7.5 slots each here.
constexpr int32_t kWaitChunk = 3;     // mean chunk size from which T = 64 waits
__host__ __device__ constexpr bool wait_for_mapping(int32_t value_bytes, int32_t block_dim,
                                                    int32_t n_rows, int64_t n_slots,
                                                    int32_t n_groups, int32_t n_heavy) {
  if (n_groups <= 0) return false;
  if (n_heavy > 0) {
    const int64_t small = value_bytes == 8   ? (block_dim == 64 ? 950000 : 0)
                          : block_dim == 64  ? (value_bytes == 4 ? 1900000 : 0)
                          : block_dim == 128 ? 1550000
                                             : 800000;
    if (n_slots <= small) return true;
  }
  if (value_bytes != 4 || block_dim != 64) return false;
  const bool full_groups = n_rows > int64_t(n_groups - 1) * block_dim;
  return !full_groups && n_slots >= kWaitChunk * int64_t(n_groups) * block_dim;
}

}  // namespace argcsr
