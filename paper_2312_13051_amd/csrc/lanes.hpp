// Sums across the lanes of a wave without LDS permutes, loops over registers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>

namespace {

// Values of the lanes L ^ o of a wave, by VALU lane moves instead of LDS
// permutes (which __shfl_xor takes): o = 32 and 16 by the half and row swaps of
// CDNA4, 8 .. 1 by DPP. The sums below add the same pairs in the same order,
// so results keep their bits. The panel's column sums kept the LDS pipe busy
// beside the loads; panel time with permutes -> without: FP32 order 96, 1,024
// matrices 1.75 -> 1.49 ms; 400, 4,608: 121.8 -> 113.3 ms (5.75 TB/s of the 6.2
// that a read reaches on this device); FP64 400, 2,304: 126.8 -> 117.0 ms; 1024,
// 256: 196.5 -> 173.8 ms.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
// v of lane L ^ O, O = 8, 4, 2 or 1
template <int O, typename T>
__device__ __forceinline__ T lane_xor(T v) {
  if constexpr (O == 8) return dpp_mov<0x128>(v);                         // row_ror:8
  else if constexpr (O == 4) return dpp_mov<0x1B>(dpp_mov<0x141>(v));    // row_half_mirror, quad_perm [3,2,1,0]
  else if constexpr (O == 2) return dpp_mov<0x4E>(v);                     // quad_perm [2,3,0,1]
  else return dpp_mov<0xB1>(v);                                           // quad_perm [1,0,3,2]
}
// lanes with bit O of L clear: a(L) + a(L ^ O); set: b(L) + b(L ^ O); O = 32 or 16
template <int O>
__device__ __forceinline__ uint2 lane_swap(uint32_t a, uint32_t b) {
  const auto r = O == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                         : __builtin_amdgcn_permlane16_swap(a, b, false, false);
  return make_uint2(r[0], r[1]);
}
template <int O>
__device__ __forceinline__ float fold(float a, float b) {
  const uint2 r = lane_swap<O>(__float_as_uint(a), __float_as_uint(b));
  return __uint_as_float(r.x) + __uint_as_float(r.y);
}
template <int O>
__device__ __forceinline__ double fold(double a, double b) {
  const uint2 l = lane_swap<O>(uint32_t(__double2loint(a)), uint32_t(__double2loint(b)));
  const uint2 h = lane_swap<O>(uint32_t(__double2hiint(a)), uint32_t(__double2hiint(b)));
  return __hiloint2double(int(h.x), int(l.x)) + __hiloint2double(int(h.y), int(l.y));
}

// max(v of L, v of L ^ O), O = 32 or 16
template <int O>
__device__ __forceinline__ double fold_max(double v) {
  const uint2 l = lane_swap<O>(uint32_t(__double2loint(v)), uint32_t(__double2loint(v)));
  const uint2 h = lane_swap<O>(uint32_t(__double2hiint(v)), uint32_t(__double2hiint(v)));
  return fmax(__hiloint2double(int(h.x), int(l.x)), __hiloint2double(int(h.y), int(l.y)));
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  v = fold<32>(v, v);
  v = fold<16>(v, v);
  v += lane_xor<8>(v);
  v += lane_xor<4>(v);
  v += lane_xor<2>(v);
  v += lane_xor<1>(v);
  return v;
}

// f(integral_constant<0>) ... f(integral_constant<N - 1>): loops over registers
// whose index has to be a constant from the start
template <int... I, typename F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F &&f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F &&f) {
  unrolled(std::make_integer_sequence<int, N>{}, f);
}

}  // namespace
