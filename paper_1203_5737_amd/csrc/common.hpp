// Shared helpers of libargcsr: status reporting (status.hpp) and wave-level
// device primitives.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <string>

#include "status.hpp"

namespace argcsr {

// XCD-aware block remap: hardware dispatches consecutive workgroups round-robin
// over the 8 XCDs; give every XCD a contiguous range of logical blocks so that
// neighbouring groups (which gather neighbouring x lines) share one L2.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb) {
  constexpr uint32_t kXcd = 8;
  const uint32_t q = nb / kXcd, r = nb % kXcd;
  const uint32_t x = b % kXcd, i = b / kXcd;
  return x * q + (x < r ? x : r) + i;
}

// Orders this wave's LDS accesses (a wave executes its LDS operations in
// issue order; the fences stop the compiler from moving accesses across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// The pointer stored in `member` (of a record in memory), as a T* known to
// point to global memory: it is read as a pointer of the global address space.
// Read as it is declared it would be a generic pointer, and its loads and
// stores FLAT accesses, which count as LDS accesses too and are never scalar
// loads.
template <typename T, typename M>
__device__ __forceinline__ T* global_ptr(M* const& member) {
  using Global = __attribute__((address_space(1))) T*;
  return (T*)*reinterpret_cast<const Global*>(&member);
}

template <typename T>
__device__ __forceinline__ T wave_uniform(T v) {
  return __builtin_amdgcn_readfirstlane(v);
}

// One data-parallel-primitive step: v of the lane that CTRL names, `old` in
// lanes whose row ROWS leaves out or that have no such lane.  These steps run
// in the vector ALU (a few cycles each); a shuffle goes through LDS.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int dpp_move(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
constexpr int kDppRowShr = 0x110;      // + n: the lane n before, within 16 lanes
constexpr int kDppRowBcast15 = 0x142;  // lane 15 of the 16 lanes before
constexpr int kDppRowBcast31 = 0x143;  // lane 31

// Inclusive wave-wide prefix sum and maximum.  Every lane must be active.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += dpp_move<kDppRowShr + 1>(0, v);
  v += dpp_move<kDppRowShr + 2>(0, v);
  v += dpp_move<kDppRowShr + 4>(0, v);
  v += dpp_move<kDppRowShr + 8>(0, v);
  v += dpp_move<kDppRowBcast15, 0xa>(0, v);
  v += dpp_move<kDppRowBcast31, 0xc>(0, v);
  return v;
}

__device__ __forceinline__ int wave_inclusive_max(int v) {
  constexpr int kLow = INT32_MIN;
  auto up = [](int x, int y) { return x > y ? x : y; };
  v = up(v, dpp_move<kDppRowShr + 1>(kLow, v));
  v = up(v, dpp_move<kDppRowShr + 2>(kLow, v));
  v = up(v, dpp_move<kDppRowShr + 4>(kLow, v));
  v = up(v, dpp_move<kDppRowShr + 8>(kLow, v));
  v = up(v, dpp_move<kDppRowBcast15, 0xa>(kLow, v));
  v = up(v, dpp_move<kDppRowBcast31, 0xc>(kLow, v));
  return v;
}

// Wave-wide sum (modulo 2^32) and maximum, the same in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  return uint32_t(__builtin_amdgcn_readlane(wave_inclusive_scan(int(v)), 63));
}

__device__ __forceinline__ int wave_max(int v) {
  return __builtin_amdgcn_readlane(wave_inclusive_max(v), 63);
}

}  // namespace argcsr
