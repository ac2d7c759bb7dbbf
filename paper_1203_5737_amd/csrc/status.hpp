// Status reporting of libargcsr, for host code that holds no device code.
#pragma once

#include <hip/hip_runtime.h>

#include "argcsr.h"

namespace argcsr {

// Records a message for argcsr_last_error() and returns `code`.
int fail(int code, const char* fmt, ...);
void clear_error();

#define ARGCSR_HIP(call)                                                       \
  do {                                                                         \
    hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess)                                                      \
      return ::argcsr::fail(ARGCSR_EHIP, "%s failed: %s (%s:%d)", #call,       \
                            hipGetErrorString(e_), __FILE__, __LINE__);        \
  } while (0)

}  // namespace argcsr
