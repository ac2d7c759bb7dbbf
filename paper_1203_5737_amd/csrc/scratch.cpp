#include "scratch.hpp"

#include <algorithm>
#include <mutex>

#include "capture.hpp"

namespace argcsr {
namespace {

constexpr int kMaxDevices = 64;

struct Block {
  void* p;
  size_t bytes;
};

// Blocks are kept in fixed arrays: nothing here allocates host memory, so
// neither a destructor nor a C entry can throw.
struct Cache {
  std::mutex mu;
  Block blocks[DeviceScratch::kKeepBlocks + 1];   // oldest first; guarded by mu
  int n = 0;
  size_t bytes = 0;               // of blocks

  Block take(int i) {
    const Block b = blocks[i];
    std::copy(blocks + i + 1, blocks + n, blocks + i);
    --n;
    bytes -= b.bytes;
    return b;
  }
};
// (a mutex and plain words: constant to construct, nothing to destroy)
Cache g_caches[kMaxDevices];

// Sizes are rounded so that calls of about the same size share blocks.
size_t rounded(size_t bytes) {
  const size_t step = bytes > (size_t(4) << 20) ? size_t(2) << 20 : size_t(64) << 10;
  return (std::max<size_t>(bytes, 1) + step - 1) / step * step;
}

// Frees what a cache holds.
void empty(Cache& c) {
  Block drop[DeviceScratch::kKeepBlocks + 1];
  int n_drop = 0;
  {
    std::lock_guard<std::mutex> lock(c.mu);
    while (c.n > 0) drop[n_drop++] = c.take(c.n - 1);
  }
  const RelaxedCapture relaxed;
  for (int i = 0; i < n_drop; ++i) (void)hipFree(drop[i].p);
}

}  // namespace

int DeviceScratch::trim() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(ARGCSR_EHIP, "no current device");
  empty(g_caches[dev]);
  return ARGCSR_OK;
}

int DeviceScratch::alloc(size_t bytes, hipStream_t s) {
  release();
  int rc = refuse_capture(s);
  if (rc) return rc;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(ARGCSR_EHIP, "no current device");
  const size_t want = rounded(bytes);
  Cache& c = g_caches[dev];
  {
    std::lock_guard<std::mutex> lock(c.mu);
    // the smallest block that fits, but none four times too large
    int best = -1;
    for (int i = 0; i < c.n; ++i) {
      const size_t b = c.blocks[i].bytes;
      if (b >= want && b / 4 <= want && (best < 0 || b < c.blocks[best].bytes)) best = i;
    }
    if (best >= 0) {
      const Block b = c.take(best);
      ptr_ = b.p;
      bytes_ = b.bytes;
    }
  }
  if (!ptr_) {
    const RelaxedCapture relaxed;
    hipError_t e = hipMalloc(&ptr_, want);
    if (e == hipErrorOutOfMemory) {
      empty(c);
      e = hipMalloc(&ptr_, want);
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      ptr_ = nullptr;
      return fail(e == hipErrorOutOfMemory ? ARGCSR_ENOMEM : ARGCSR_EHIP,
                  "device scratch of %zu bytes could not be allocated: %s", bytes,
                  hipGetErrorString(e));
    }
    bytes_ = want;
  }
  device_ = dev;
  stream_ = s;
  idle_ = false;
  return ARGCSR_OK;
}

void DeviceScratch::release() {
  if (!ptr_) return;
  void* p = ptr_;
  ptr_ = nullptr;
  // an owner that left early may have work queued that uses the block; if
  // waiting fails, the block is not handed out again
  if (!idle_) {
    const RelaxedCapture relaxed;
    if (hipStreamSynchronize(stream_) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
  }
  Cache& c = g_caches[device_];
  Block drop[DeviceScratch::kKeepBlocks + 1];
  int n_drop = 0;
  {
    std::lock_guard<std::mutex> lock(c.mu);
    c.blocks[c.n++] = Block{p, bytes_};
    c.bytes += bytes_;
    while (c.bytes > kKeepBytes || c.n > kKeepBlocks) drop[n_drop++] = c.take(0);
  }
  if (n_drop > 0) {
    const RelaxedCapture relaxed;
    for (int i = 0; i < n_drop; ++i) (void)hipFree(drop[i].p);
  }
}

}  // namespace argcsr

extern "C" int argcsr_trim_scratch(void) {
  argcsr::clear_error();
  return argcsr::DeviceScratch::trim();
}
