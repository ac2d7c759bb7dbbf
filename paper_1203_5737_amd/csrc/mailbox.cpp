#include "mailbox.hpp"

#include <hip/hip_runtime.h>

#include <mutex>

#include "capture.hpp"

namespace argcsr {
namespace {

constexpr int kSlots = 256;
constexpr size_t kSlotBytes = sizeof(int64_t) * Mailbox::kWords;
// visible to every device and written through to the host
constexpr unsigned kFlags = hipHostMallocMapped | hipHostMallocPortable | hipHostMallocCoherent;

std::mutex g_mu;
int64_t* g_block = nullptr;           // kSlots slots, guarded by g_mu
int64_t* g_free[kSlots];              // free ones, the first g_n_free; guarded by g_mu
int g_n_free = 0;

}  // namespace

int Mailbox::init(hipStream_t s) {
  const int rc = refuse_capture(s);
  if (rc) return rc;
  {
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_block) {
      const RelaxedCapture relaxed;
      void* p = nullptr;
      if (hipHostMalloc(&p, kSlots * kSlotBytes, kFlags) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ARGCSR_ENOMEM, "pinned result slots could not be allocated");
      }
      g_block = static_cast<int64_t*>(p);
      for (int i = kSlots - 1; i >= 0; --i) g_free[g_n_free++] = g_block + i * kWords;
    }
    if (g_n_free > 0) host_ = g_free[--g_n_free];
  }
  if (!host_) {
    const RelaxedCapture relaxed;
    void* p = nullptr;
    if (hipHostMalloc(&p, kSlotBytes, kFlags) != hipSuccess) {
      (void)hipGetLastError();
      return fail(ARGCSR_ENOMEM, "pinned result slot could not be allocated");
    }
    host_ = static_cast<int64_t*>(p);
    own_ = true;
  }
  void* d = nullptr;
  if (hipHostGetDevicePointer(&d, host_, 0) != hipSuccess)
    return fail(ARGCSR_EHIP, "pinned result slot is not mapped on this device");
  dev_ = static_cast<int64_t*>(d);
  stream_ = s;
  idle_ = false;
  for (int i = 0; i < kWords; ++i) static_cast<volatile int64_t*>(host_)[i] = 0;
  return ARGCSR_OK;
}

Mailbox::~Mailbox() {
  if (!host_) return;
  // an owner that left early may have kernels queued that write the slot
  if (!idle_) {
    const RelaxedCapture relaxed;
    if (hipStreamSynchronize(stream_) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
  }
  if (own_) {
    const RelaxedCapture relaxed;
    (void)hipHostFree(host_);
    return;
  }
  std::lock_guard<std::mutex> lock(g_mu);
  g_free[g_n_free++] = host_;
}

}  // namespace argcsr
