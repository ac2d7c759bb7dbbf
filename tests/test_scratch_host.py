"""CPU: the library's pinned result slots and its cache of device scratch
(host bookkeeping only), built with g++ under AddressSanitizer and
UndefinedBehaviorSanitizer against a stand-in for the HIP calls they make.
The stand-in hands out host memory, keeps the list of calls, and fails where
the driver tells it to."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1203_5737_amd", "csrc")

HIP = r"""
#pragma once
#include <cstddef>
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorCapture = 900,
                  hipErrorUnknown = 999 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal,
                            hipStreamCaptureModeRelaxed };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
typedef struct ihipStream_t* hipStream_t;
constexpr unsigned hipHostMallocMapped = 2, hipHostMallocPortable = 1,
                   hipHostMallocCoherent = 0x40000000;
hipError_t hipGetDevice(int*);
hipError_t hipMalloc(void**, size_t);
hipError_t hipFree(void*);
hipError_t hipHostMalloc(void**, size_t, unsigned);
hipError_t hipHostFree(void*);
hipError_t hipHostGetDevicePointer(void**, void*, unsigned);
hipError_t hipStreamSynchronize(hipStream_t);
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus*);
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*);
hipError_t hipGetLastError();
inline const char* hipGetErrorString(hipError_t) { return ""; }
"""

COMMON = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <memory>
#include <string>
#include <vector>
#include "mailbox.hpp"
#include "scratch.hpp"
#include "status.hpp"

static std::map<void*, size_t> g_dev, g_pinned;      // live allocations
static int g_syncs, g_mallocs, g_frees;
static hipError_t g_sync_result = hipSuccess, g_malloc_result = hipSuccess;
static size_t g_room = size_t(1) << 40;              // device memory there is

static hipStream_t g_capturing = nullptr;            // a stream that is capturing a graph
static bool g_global = false;                        // another thread is, in the global mode
static hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
static int g_refused;                                // calls that mode forbade
static bool forbidden() {
  const bool no = g_global && g_mode == hipStreamCaptureModeGlobal;
  g_refused += no;
  return no;
}

hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = s && s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, g_mode);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
static hipError_t hip_malloc(void** p, size_t n) {
  if (forbidden()) return hipErrorCapture;
  ++g_mallocs;
  if (g_malloc_result != hipSuccess) return g_malloc_result;
  size_t used = 0;
  for (auto& b : g_dev) used += b.second;
  if (used + n > g_room) return hipErrorOutOfMemory;
  *p = std::malloc(16);                              // never touched: its size is only noted
  g_dev[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (forbidden()) return hipErrorCapture;
  if (!g_dev.erase(p)) std::abort();
  ++g_frees;
  std::free(p);
  return hipSuccess;
}
static hipError_t hip_host_malloc(void** p, size_t n, unsigned) {
  if (forbidden()) return hipErrorCapture;
  *p = std::malloc(n);
  g_pinned[*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  if (forbidden()) return hipErrorCapture;
  if (!g_pinned.erase(p)) std::abort();
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  if (forbidden()) return hipErrorCapture;
  ++g_syncs;
  return g_sync_result;
}
hipError_t hipGetLastError() { return hipSuccess; }
namespace argcsr {
int fail(int code, const char*, ...) { return code; }
void clear_error() {}
}  // namespace argcsr
using argcsr::DeviceScratch;
using argcsr::Mailbox;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
"""

PLAIN = r"""
hipError_t hipMalloc(void** p, size_t n) { return hip_malloc(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) { return hip_host_malloc(p, n, f); }
"""

SLOTS = PLAIN + r"""
int main() {
  hipStream_t s = reinterpret_cast<hipStream_t>(0x10);
  int64_t* slot;
  {                                     // waited for by its owner
    Mailbox m;
    CHECK(m.init(s) == ARGCSR_OK);
    slot = m.device();
    slot[3] = 7;
    CHECK(m.word(3) == 7);
    m.idle();
  }
  CHECK(g_syncs == 0);
  {                                     // an owner that leaves early: the slot goes back only
    Mailbox m;                          // when its stream has been waited for, and starts at zero
    CHECK(m.init(s) == ARGCSR_OK && m.device() == slot && m.word(3) == 0);
  }
  CHECK(g_syncs == 1);
  {                                     // a stream that cannot be waited for: the slot is lost
    Mailbox m;
    CHECK(m.init(s) == ARGCSR_OK && m.device() == slot);
    g_sync_result = hipErrorUnknown;
  }
  g_sync_result = hipSuccess;
  std::map<int64_t*, int> seen;
  std::vector<std::unique_ptr<Mailbox>> many;
  for (int i = 0; i < 300; ++i) {       // past the block's 256 slots: a block each
    many.emplace_back(new Mailbox);
    CHECK(many.back()->init(s) == ARGCSR_OK);
    CHECK(many.back()->device() != slot && seen[many.back()->device()]++ == 0);
    many.back()->device()[Mailbox::kWords - 1] = i;
    many.back()->idle();
  }
  CHECK(g_pinned.size() == 1 + 300 - 255);
  for (int i = 0; i < 300; ++i) CHECK(many[size_t(i)]->word(Mailbox::kWords - 1) == i);
  many.clear();
  CHECK(g_pinned.size() == 1 && g_syncs == 2);
  std::puts("ok");
  std::fflush(stdout);
  std::_Exit(0);                        // the block of slots is kept until the process ends
}
"""


BLOCKS = PLAIN + r"""
constexpr size_t kMB = size_t(1) << 20;
static size_t live() {
  size_t n = 0;
  for (auto& b : g_dev) n += b.second;
  return n;
}
int main() {
  hipStream_t s = reinterpret_cast<hipStream_t>(0x10);
  void* first;
  {                                     // a block comes back for a call of its size
    DeviceScratch a, b;
    CHECK(a.alloc(100 * kMB, s) == ARGCSR_OK && b.alloc(100 * kMB, s) == ARGCSR_OK);
    first = a.ptr();
    CHECK(first != b.ptr());
    a.idle();
    a.release();
    CHECK(g_syncs == 0);
    DeviceScratch c;
    CHECK(c.alloc(100 * kMB - 5, s) == ARGCSR_OK && c.ptr() == first && g_mallocs == 2);
    c.release();                        // its owner has not said idle
    CHECK(g_syncs == 1);
    DeviceScratch d;
    CHECK(d.alloc(24 * kMB, s) == ARGCSR_OK && d.ptr() != first);   // four times too large
    d.idle();
    b.idle();
  }
  CHECK(g_dev.size() == 3 && g_frees == 0);
  {                                     // more blocks than are kept: the oldest go
    std::vector<std::unique_ptr<DeviceScratch>> many;
    for (int i = 0; i < DeviceScratch::kKeepBlocks; ++i) {
      many.emplace_back(new DeviceScratch);
      CHECK(many.back()->alloc((5 + size_t(i) / 8) * kMB, s) == ARGCSR_OK);
      many.back()->idle();
    }
  }
  CHECK(int(g_dev.size()) == DeviceScratch::kKeepBlocks && g_dev.count(first) == 0);
  {                                     // more bytes than are kept
    DeviceScratch a;
    CHECK(a.alloc(DeviceScratch::kKeepBytes - 8 * kMB, s) == ARGCSR_OK);
    a.idle();
  }
  CHECK(live() <= DeviceScratch::kKeepBytes && g_dev.size() == 2);
  {                                     // out of memory: what is cached goes, then again
    g_room = live() + kMB;
    DeviceScratch a;
    CHECK(a.alloc(64 * kMB, s) == ARGCSR_OK && g_dev.size() == 1);
    DeviceScratch b;
    CHECK(b.alloc(DeviceScratch::kKeepBytes, s) == ARGCSR_ENOMEM && !b.ptr());
    g_room = size_t(1) << 40;
    a.idle();
  }
  CHECK(g_dev.size() == 1);
  {                                     // given back on request, what is in use is not
    DeviceScratch a, b;
    CHECK(a.alloc(64 * kMB, s) == ARGCSR_OK && b.alloc(64 * kMB, s) == ARGCSR_OK);
    a.idle();
    a.release();
    CHECK(argcsr_trim_scratch() == ARGCSR_OK && g_dev.size() == 1 && g_dev.count(b.ptr()) == 1);
    b.idle();
  }
  CHECK(g_dev.size() == 1);
  {                                     // any other failure is no lack of memory: the cache stays
    g_malloc_result = hipErrorUnknown;
    DeviceScratch a;
    CHECK(a.alloc(256 * kMB, s) == ARGCSR_EHIP && !a.ptr());
    g_malloc_result = hipSuccess;
    CHECK(g_dev.size() == 1);
  }
  {                                     // another thread captures in the global mode: blocks are
    g_global = true;                    // taken, waited for, kept and freed as before
    const int frees = g_frees;
    DeviceScratch a, b, c;
    CHECK(a.alloc(64 * kMB, s) == ARGCSR_OK && b.alloc(DeviceScratch::kKeepBytes, s) == ARGCSR_OK);
    a.release();
    CHECK(c.alloc(64 * kMB, s) == ARGCSR_OK);
    c.release();
    b.release();
    CHECK(g_dev.size() == 1 && g_frees == frees + 1);
    Mailbox m;
    CHECK(m.init(s) == ARGCSR_OK);
    CHECK(g_refused == 0 && g_mode == hipStreamCaptureModeGlobal);
    g_global = false;
  }
  {                                     // the stream itself is capturing: refused, nothing taken
    g_capturing = s;
    const size_t blocks = g_dev.size();
    const int syncs = g_syncs;
    DeviceScratch a;
    Mailbox m;
    CHECK(a.alloc(64 * kMB, s) == ARGCSR_EHIP && m.init(s) == ARGCSR_EHIP);
    CHECK(!a.ptr() && g_dev.size() == blocks && g_syncs == syncs);
    g_capturing = nullptr;
  }
  {                                     // a stream that cannot be waited for: the block is lost
    DeviceScratch a, b;
    CHECK(a.alloc(kMB, s) == ARGCSR_OK);
    void* p = a.ptr();
    g_sync_result = hipErrorUnknown;
    a.release();
    g_sync_result = hipSuccess;
    CHECK(b.alloc(kMB, s) == ARGCSR_OK && b.ptr() != p);
    b.idle();
  }
  std::puts("ok");
  std::fflush(stdout);
  std::_Exit(0);
}
"""

# every allocation of host memory by the two files fails: nothing throws, in a
# destructor or out of a call
NO_HOST_MEMORY = r"""
#include <new>
static bool g_no_memory = false;
void* operator new(size_t n) {
  if (g_no_memory) throw std::bad_alloc();
  return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// the stand-in's own lists may allocate
struct Allow {
  bool was = g_no_memory;
  Allow() { g_no_memory = false; }
  ~Allow() { g_no_memory = was; }
};
hipError_t hipMalloc(void** p, size_t n) { Allow a; return hip_malloc(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) { Allow a; return hip_host_malloc(p, n, f); }

int main() {
  hipStream_t s = reinterpret_cast<hipStream_t>(0x10);
  g_no_memory = true;
  bool ok = true;
  for (int round = 0; round < 2; ++round) {
    DeviceScratch b[DeviceScratch::kKeepBlocks + 4];
    for (auto& x : b) {
      ok = ok && x.alloc(5 << 20, s) == ARGCSR_OK;
      x.idle();
    }
    Mailbox m[300];
    for (auto& x : m) {
      ok = ok && x.init(s) == ARGCSR_OK;
      x.idle();
    }
    for (auto& x : b) x.release();
    g_room = 0;                          // empties the cache
    ok = ok && b[0].alloc(1 << 30, s) == ARGCSR_ENOMEM;
    g_room = size_t(1) << 40;
  }
  g_no_memory = false;
  CHECK(ok && g_dev.empty());
  std::puts("ok");
  std::fflush(stdout);
  std::_Exit(0);
}
"""


def run(tmp_path, main):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    src = tmp_path / "drv.cpp"
    src.write_text(COMMON + main)
    exe = tmp_path / "drv"
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", str(tmp_path), "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), str(src),
                    os.path.join(CSRC, "mailbox.cpp"), os.path.join(CSRC, "scratch.cpp"),
                    "-o", str(exe)], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and "ok" in r.stdout, (r.returncode, r.stdout, r.stderr[-3000:])


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_result_slots_wait_for_their_stream(tmp_path):
    run(tmp_path, SLOTS)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_device_scratch_cache(tmp_path):
    """Reuse, eviction by number and by size, lack of memory, other failures,
    and graph capture by this and by another thread."""
    run(tmp_path, BLOCKS)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_host_allocation_throws(tmp_path):
    run(tmp_path, NO_HOST_MEMORY)
