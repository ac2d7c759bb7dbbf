// Device scratch of the calls that wait for their stream before they return
// (planning, conversion, binning).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace argcsr {

// One block of device memory on the current device, held from alloc to
// destruction.  Blocks come from a cache per device and go back to it once
// the stream they were used on has been waited for: by the owner, who then
// says idle(), or else by the destructor.  A block in the cache is therefore
// unused on the device and may go to any stream and thread next.  (A
// stream-ordered allocation needs no wait, but its hipFreeAsync takes 8 to
// 16 us on the host, three times per conversion: without it the conversion of
// the power-law matrix of 10^6 rows went from 210 to 184 us.)  The cache keeps
// at most kKeepBytes and kKeepBlocks per device -- the scratch of planning and
// converting a matrix of about 9*10^7 rows, at 22 bytes a row and what the
// fill's list of long tiles takes -- and frees the oldest blocks beyond that
// (a larger matrix allocates again on each call); when the device is out of
// memory everything cached is freed and the allocation tried again.
class DeviceScratch {
 public:
  static constexpr size_t kKeepBytes = size_t(2) << 30;
  static constexpr int kKeepBlocks = 16;
  DeviceScratch() = default;
  DeviceScratch(const DeviceScratch&) = delete;
  DeviceScratch& operator=(const DeviceScratch&) = delete;
  ~DeviceScratch() { release(); }
  int alloc(size_t bytes, hipStream_t s);    // ARGCSR_OK or ARGCSR_ENOMEM
  void* ptr() const { return ptr_; }
  // the owner has waited for the stream and uses the block no more on it, or
  // waits again before the block goes
  void idle() { idle_ = true; }
  void release();
  // frees what the current device's cache holds (argcsr_trim_scratch)
  static int trim();

 private:
  void* ptr_ = nullptr;
  size_t bytes_ = 0;
  int device_ = -1;
  hipStream_t stream_ = nullptr;
  bool idle_ = false;
};

}  // namespace argcsr
