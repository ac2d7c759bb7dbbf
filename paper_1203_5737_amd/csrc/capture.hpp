// Graph capture, as seen by the calls that wait for their stream (planning,
// conversion, staging, binning) and hold memory between calls.
#pragma once

#include "status.hpp"

namespace argcsr {

// Refuses, before anything is queued, a call that waits for a stream that
// is capturing a graph.  Its kernels would be recorded and not run, the wait
// fails, and the memory they name could never be used again.
inline int refuse_capture(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();            // not known: the wait itself will tell
    return ARGCSR_OK;
  }
  if (st == hipStreamCaptureStatusNone) return ARGCSR_OK;
  return fail(ARGCSR_EHIP, "the call waits for its stream, which is capturing a graph");
}

// While this lives, the calling thread may allocate, free and wait although
// another thread captures a graph in the global mode, which forbids these
// calls to every thread; none of them concerns that graph.
class RelaxedCapture {
 public:
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  RelaxedCapture(const RelaxedCapture&) = delete;
  RelaxedCapture& operator=(const RelaxedCapture&) = delete;

 private:
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

}  // namespace argcsr
