// Helpers of the kernels that march in registers, one lane per column (gfx950): values of the
// neighbouring lanes, wave-uniform table reads and compile-time indices.  Included by the
// kernel sources only.
#pragma once

#include "lbm_ch_device.h"

#include <type_traits>

namespace lbmch {
namespace {

// The value of the lane to the west (x - 1) and to the east (x + 1): whole-wave shifts by
// one lane; the lane at the end gets 0.
__device__ __forceinline__ int west_i(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int east_i(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float west(float v) {
  return __builtin_bit_cast(float, west_i(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ float east(float v) {
  return __builtin_bit_cast(float, east_i(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double west(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)west_i((int)(uint32_t)u), hi = (uint32_t)west_i((int)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double east(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)east_i((int)(uint32_t)u), hi = (uint32_t)east_i((int)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// A non-temporal load (CP_NT).
__device__ __forceinline__ float ldb_nt(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, CP_NT));
}

// A table read at a wave-uniform index through the scalar cache (never written while a
// step runs).
__device__ __forceinline__ float ld_uniform(const float* p, int i) {
  return ((const __attribute__((address_space(4))) float*)(uintptr_t)p)[i];
}

template <int N>
using ic = std::integral_constant<int, N>;

}  // namespace
}  // namespace lbmch
