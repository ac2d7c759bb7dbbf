#include "scratch.hpp"

#include <algorithm>
#include <mutex>
#include <vector>

#include "capture.hpp"

namespace argcsr {
namespace {

constexpr int kMaxDevices = 64;

struct Block {
  void* p;
  size_t bytes;
};

struct Cache {
  std::mutex mu;
  std::vector<Block> blocks;      // oldest first; guarded by mu
  size_t bytes = 0;               // of blocks
};

// Never destroyed: the runtime may be gone when static objects are.
Cache& cache_of(int device) {
  static Cache* const caches = new Cache[kMaxDevices];
  return caches[device];
}

// Sizes are rounded so that calls of about the same size share blocks.
size_t rounded(size_t bytes) {
  const size_t step = bytes > (size_t(4) << 20) ? size_t(2) << 20 : size_t(64) << 10;
  return (std::max<size_t>(bytes, 1) + step - 1) / step * step;
}

}  // namespace

int DeviceScratch::alloc(size_t bytes, hipStream_t s) {
  release();
  int rc = refuse_capture(s);
  if (rc) return rc;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(ARGCSR_EHIP, "no current device");
  const size_t want = rounded(bytes);
  Cache& c = cache_of(dev);
  std::vector<Block> drop;
  {
    std::lock_guard<std::mutex> lock(c.mu);
    // the smallest block that fits, but none four times too large
    int best = -1;
    for (int i = 0; i < int(c.blocks.size()); ++i) {
      const size_t b = c.blocks[size_t(i)].bytes;
      if (b >= want && b / 4 <= want && (best < 0 || b < c.blocks[size_t(best)].bytes)) best = i;
    }
    if (best >= 0) {
      ptr_ = c.blocks[size_t(best)].p;
      bytes_ = c.blocks[size_t(best)].bytes;
      c.bytes -= bytes_;
      c.blocks.erase(c.blocks.begin() + best);
    }
  }
  if (!ptr_) {
    const RelaxedCapture relaxed;
    hipError_t e = hipMalloc(&ptr_, want);
    if (e == hipErrorOutOfMemory) {
      {
        std::lock_guard<std::mutex> lock(c.mu);
        drop.swap(c.blocks);
        c.bytes = 0;
      }
      for (const Block& b : drop) (void)hipFree(b.p);
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
  Cache& c = cache_of(device_);
  std::vector<Block> drop;
  {
    std::lock_guard<std::mutex> lock(c.mu);
    c.blocks.push_back(Block{p, bytes_});
    c.bytes += bytes_;
    while (c.bytes > kKeepBytes || int(c.blocks.size()) > kKeepBlocks) {
      drop.push_back(c.blocks.front());
      c.bytes -= c.blocks.front().bytes;
      c.blocks.erase(c.blocks.begin());
    }
  }
  if (!drop.empty()) {
    const RelaxedCapture relaxed;
    for (const Block& b : drop) (void)hipFree(b.p);
  }
}

}  // namespace argcsr
