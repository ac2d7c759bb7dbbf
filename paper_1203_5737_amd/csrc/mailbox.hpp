// Small results a kernel hands to the host: 64-byte slots of mapped pinned
// host memory that kernels write themselves, so that a call which must know
// a size or a flag waits for its stream once, with no copy queued behind the
// kernels (a copy into pageable memory and its staging cost about 15 us more
// than the store).  Kernels write a slot with plain vector stores; the host
// reads it after it has waited for the stream.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace argcsr {

// One slot, held from init to destruction; its words start at zero.
// Slots come from one 16-KiB block, taken on first use and kept until the
// process ends; past its 256 slots a caller gets a block of its own.  A slot
// goes back once the stream it was used on has been waited for: by the owner,
// who then says idle(), or else by the destructor; one that cannot be waited
// for is not handed out again.  Safe with any number of threads, streams and
// devices.
class Mailbox {
 public:
  static constexpr int kWords = 8;
  Mailbox() = default;
  Mailbox(const Mailbox&) = delete;
  Mailbox& operator=(const Mailbox&) = delete;
  ~Mailbox();
  int init(hipStream_t s);                   // ARGCSR_OK or a status code
  int64_t* device() const { return dev_; }
  // the host's view; read it after waiting for the writing stream
  int64_t word(int i) const { return static_cast<volatile const int64_t*>(host_)[i]; }
  // the owner has waited for the stream and queues no more kernels that
  // write the slot
  void idle() { idle_ = true; }

 private:
  int64_t* host_ = nullptr;
  int64_t* dev_ = nullptr;
  hipStream_t stream_ = nullptr;
  bool own_ = false;
  bool idle_ = true;                         // until a kernel can know the slot
};

}  // namespace argcsr
