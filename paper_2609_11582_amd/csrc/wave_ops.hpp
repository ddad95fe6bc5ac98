// Exchanges between the lanes of a wave on the VALU (DPP moves and the row swaps of gfx950), for the decode kernels.
#pragma once

#include "okvq_device.hpp"

namespace okvq {

// lane l <- lane l ^ 8 within each row of 16 lanes (DPP row rotate by 8)
constexpr int kRowRor8 = 0x128;
__device__ __forceinline__ float fswap8(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kRowRor8, 0xf, 0xf, false));
}
// Pairwise combination of lanes l and l ^ 16 (or l ^ 32) with the VALU row swaps of gfx950
// (v_permlane16_swap / v_permlane32_swap): swapping a register with a copy of itself leaves the
// lane's own value in one result and its partner's in the other, so a symmetric op of the two
// results is the pair's value in both lanes, with no LDS-pipe shuffle. The copy is made opaque:
// given the same value twice, the compiler folds the two results into one.
__device__ __forceinline__ uint32_t opaque_copy(uint32_t v) {
  __asm__ volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ void swap16(uint32_t v, uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, opaque_copy(v), false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap32(uint32_t v, uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, opaque_copy(v), false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ float sum16(float v) {
  uint32_t a, b;
  swap16(__builtin_bit_cast(uint32_t, v), a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float sum32(float v) {
  uint32_t a, b;
  swap32(__builtin_bit_cast(uint32_t, v), a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float max16(float v) {
  uint32_t a, b;
  swap16(__builtin_bit_cast(uint32_t, v), a, b);
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float max32(float v) {
  uint32_t a, b;
  swap32(__builtin_bit_cast(uint32_t, v), a, b);
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
// lane ^ 4 within each row of 16
__device__ __forceinline__ float fswap4(float v) {
  const int x = __builtin_bit_cast(int, v);
  const int t = __builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0x5, false);  // banks 0, 2: lane + 4
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(t, x, 0x114, 0xf, 0xa, false));  // 1, 3: lane - 4
}
// DPP move of all lanes (0xB1: lane ^ 1, 0x4E: lane ^ 2, 0x150 + n: lane n of the row of 16)
template <int kCtrl>
__device__ __forceinline__ float fdpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
// lane ^ 16
__device__ __forceinline__ float fswap16(float v) {
  uint32_t a, b;
  swap16(__builtin_bit_cast(uint32_t, v), a, b);
  return __builtin_bit_cast(float, (lane_id() & 16) ? a : b);
}
// Lanes 0-31 and 32-63 each hold a row of 128 channels, lane l channels 4 (l & 31) .. + 3: the Hadamard
// butterflies h = 1 .. 64 in ascending order by DPP and row swaps. As LDS-pipe shuffles these and the maximum
// below were eleven dependent round trips before the first barrier of a decode: 32768 tokens 12.42 -> 11.98 us,
// 1024 tokens 10.48 -> 10.28, 8 generation steps 163 -> 160.4
__device__ __forceinline__ void hadamard_row(float (&x)[4], int lane) {
  {  // channel bits 0, 1 in lane
    const float a = x[0] + x[1], c = x[0] - x[1], d = x[2] + x[3], e = x[2] - x[3];
    x[0] = a + d;
    x[2] = a - d;
    x[1] = c + e;
    x[3] = c - e;
  }
  auto step = [&](int lb, auto&& partner) {  // channel bits 2..6 are lane bits 0..4
    const bool hi = (lane & lb) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float o = partner(x[i]);
      x[i] = hi ? o - x[i] : x[i] + o;
    }
  };
  step(1, [](float v) { return fdpp<0xB1>(v); });
  step(2, [](float v) { return fdpp<0x4E>(v); });
  step(4, [](float v) { return fswap4(v); });
  step(8, [](float v) { return fswap8(v); });
  step(16, [](float v) { return fswap16(v); });
}
// maximum over the wave, in every lane
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, fdpp<0xB1>(v));
  v = fmaxf(v, fdpp<0x4E>(v));
  v = fmaxf(v, fswap4(v));
  v = fmaxf(v, fswap8(v));
  return max32(max16(v));
}

}  // namespace okvq
