// Exchanges inside a 64-wide wave on the VALU (DPP and readlane), and a
// workgroup barrier that orders LDS alone: shared by the kernels that keep a
// whole solve on the chip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gabp {

namespace {

template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));

// Lane exchanges on the VALU (DPP); a lane without a source gets `old`.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double old, double v) {
  const uint64_t o = __builtin_bit_cast(uint64_t, old), b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp(float old, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                               __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
constexpr int kRowShr = 0x110, kBcast15 = 0x142, kBcast31 = 0x143, kWaveShl1 = 0x130, kWaveShr1 = 0x138;
__device__ __forceinline__ double readlane_r(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// A value that every lane holds alike, kept in scalar registers.
__device__ __forceinline__ double uni_r(double v) { return readlane_r(v, 0); }
// Sum over the first 16 lanes, over the wave: in scalar registers, in a fixed order.
__device__ __forceinline__ double sum16(double v) {
  v += dpp<kRowShr + 1, 0xf>(0.0, v);
  v += dpp<kRowShr + 2, 0xf>(0.0, v);
  v += dpp<kRowShr + 4, 0xf>(0.0, v);
  v += dpp<kRowShr + 8, 0xf>(0.0, v);
  return v;
}
__device__ __forceinline__ double wsum_r(double v) {
  v = sum16(v);
  v += dpp<kBcast15, 0xa>(0.0, v);
  v += dpp<kBcast31, 0xc>(0.0, v);
  return readlane_r(v, 63);
}

// Workgroup barrier ordering LDS only.
__device__ __forceinline__ void lds_barrier_r() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace

}  // namespace gabp
