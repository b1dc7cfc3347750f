// Exchanges between the 64 lanes of a wave by data-parallel primitives (no LDS round trip); every lane is active.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kp_wave {

// Lane l receives the value of lane l-1; lane 0 receives `lane0` (DPP wave shift right by one).
__device__ __forceinline__ uint32_t wave_shr1(uint32_t v, uint32_t lane0) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)lane0, (int)v, 0x138, 0xF, 0xF, false);
}

// Lane l receives the value of lane l-1; lane 0 that of lane 63 (DPP wave rotate right by one).
__device__ __forceinline__ uint32_t wave_ror1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x13C, 0xF, 0xF, true);
}

// The DPP steps of an inclusive scan over the 64 lanes: four shifts inside each row of 16, then the
// last lane of row 0/2 into row 1/3 and the last lane of the lower half into the upper half.  Lanes
// without a source read `none`.
template <int STEP> __device__ __forceinline__ uint32_t scan_src(uint32_t v, uint32_t none = 0u) {
  if (STEP == 0) return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  if (STEP == 1) return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
  if (STEP == 2) return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
  if (STEP == 3) return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
  if (STEP == 4) return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x143, 0xC, 0xF, false);                 // row_bcast:31
}

template <int STEP> __device__ __forceinline__ uint64_t scan_src64(uint64_t v) {
  return (uint64_t)scan_src<STEP>((uint32_t)v) | ((uint64_t)scan_src<STEP>((uint32_t)(v >> 32)) << 32);
}

__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v) {
  v += scan_src<0>(v); v += scan_src<1>(v); v += scan_src<2>(v);
  v += scan_src<3>(v); v += scan_src<4>(v); v += scan_src<5>(v);
  return v;
}

// The same in every lane: the sum, and the smallest value.
__device__ __forceinline__ uint32_t wave_total(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(v), 63); }
__device__ __forceinline__ uint32_t wave_least(uint32_t v) {
  auto lesser = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
  constexpr uint32_t none = 0xFFFFFFFFu;
  v = lesser(v, scan_src<0>(v, none)); v = lesser(v, scan_src<1>(v, none)); v = lesser(v, scan_src<2>(v, none));
  v = lesser(v, scan_src<3>(v, none)); v = lesser(v, scan_src<4>(v, none)); v = lesser(v, scan_src<5>(v, none));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

}  // namespace kp_wave
