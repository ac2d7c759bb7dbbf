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
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };
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

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
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
  if (!g_dev.erase(p)) std::abort();
  ++g_frees;
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::malloc(n);
  g_pinned[*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  if (!g_pinned.erase(p)) std::abort();
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_syncs; return g_sync_result; }
hipError_t hipGetLastError() { return hipSuccess; }
namespace argcsr {
int fail(int code, const char*, ...) { return code; }
void clear_error() {}
}  // namespace argcsr
using argcsr::DeviceScratch;
using argcsr::Mailbox;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
"""

SLOTS = r"""
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
