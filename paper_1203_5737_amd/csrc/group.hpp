// Conversion step 1 (grouping) on the GPU (group.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "argcsr.h"

namespace argcsr {

// Rows a workgroup of the grouping kernels handles.
constexpr int kGroupRows = 4096;

// Device words the grouping writes for the kernels after it.
struct GroupCount {
  int32_t n_groups;
  int32_t bad;           // row_ptr does not start at 0 or decreases
};

// Enqueues the grouping of n > 0 rows: `groups` (room for n entries) gets
// first_row and size of every group (offset and chunk size 0), *count the
// number of groups and whether row_ptr is malformed (the groups then still
// cover the rows, each at most block_dim of them), and the `clear_words`
// 32-bit words at `clear`, which *count is none of, are set to 0.  block_dim
// in [1, 1024].
// format ARGCSR_FORMAT_RG: groups of block_dim rows (no nonzero budget);
// region_desired (host, checked by the caller): a desiredChunkSize per region
// of region_rows rows, taken from the region of a group's first row.
// `work` is device scratch of group_work_bytes, in use until the stream has
// been waited for.
size_t group_work_bytes(int32_t n, int32_t block_dim, int32_t format, int32_t region_rows,
                        const int32_t* region_desired);
int group_on_device(int32_t n, const int32_t* row_ptr, int32_t block_dim, int32_t desired,
                    int32_t format, int32_t region_rows, const int32_t* region_desired,
                    argcsr_group_info* groups, GroupCount* count, int32_t* clear,
                    int64_t clear_words, void* work, hipStream_t s);

}  // namespace argcsr
