// Moves between the lanes of a wavefront, sums and maxima over them, on the ALUs: row shifts inside rows of 16 lanes, then
// across the rows.  (A shuffle per step goes through LDS, 100 cycles each where nothing covers them.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rdkv {

// v of the lane CTRL names; every lane has one
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, dpp_u32<CTRL>(__builtin_bit_cast(uint32_t, v)));
}
// Row and half exchanges in place (the wait states they need after a write to their operands stand in front of them): rows 1
// and 3 of a swapped with rows 0 and 2 of b; the upper half of a with the lower half of b.
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// Sum of the wavefront's two halves: of a in lanes 0..31, of b in lanes 32..63.
__device__ __forceinline__ float halves_sum(float a, float b) {
  const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}
// maximum and sum over the 16 lanes of a row, in each of them
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f32<0x128>(v));   // row_ror:8
  v = fmaxf(v, dpp_f32<0x124>(v));
  v = fmaxf(v, dpp_f32<0x122>(v));
  return fmaxf(v, dpp_f32<0x121>(v));
}
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_f32<0x128>(v);
  v += dpp_f32<0x124>(v);
  v += dpp_f32<0x122>(v);
  return v + dpp_f32<0x121>(v);
}
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
  v += dpp_u32<0x128>(v);
  v += dpp_u32<0x124>(v);
  v += dpp_u32<0x122>(v);
  return v + dpp_u32<0x121>(v);
}
__device__ __forceinline__ float sum_xor16(float v) {
  float o = v;
  swap_rows(v, o);
  return v + o;
}
// Reduction over the 16 lanes that hold the same head (lane % 4): lanes 4 apart inside a row of 16, then the rows.  No
// step goes through LDS: with two or three wavefronts per SIMD nothing covers the 100 cycles of a ds_bpermute (a chunk's
// five sums took 0.65 us).
// (A maximum that reads another lane is one instruction; out of fmaxf the compiler makes three, because it cannot tell that
// what comes from another lane is no signalling NaN.  Two wait states stand between a write to a register and its use by
// another lane.)  v: no signalling NaN
__device__ __forceinline__ float head_max(float v) {
  float o;
  asm("s_nop 1\n\t"
      "v_max_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_mov_b32 %1, %0\n\t"
      "s_nop 1\n\t"
      "v_permlane16_swap_b32 %0, %1\n\t"
      "s_nop 0\n\t"
      "v_max_f32 %0, %0, %1\n\t"
      "v_mov_b32 %1, %0\n\t"
      "s_nop 1\n\t"
      "v_permlane32_swap_b32 %0, %1\n\t"
      "s_nop 0\n\t"
      "v_max_f32 %0, %0, %1"
      : "+v"(v), "=&v"(o));
  return v;
}
// the larger of four, none a signalling NaN
__device__ __forceinline__ float max_of_four(float a, float b, float c, float d) {
  float m;
  asm("v_max3_f32 %0, %1, %2, %3\n\tv_max_f32 %0, %0, %4" : "=&v"(m) : "v"(a), "v"(b), "v"(c), "v"(d));
  return m;
}
__device__ __forceinline__ float head_sum(float v) {
  v += dpp_f32<0x124>(v);
  v += dpp_f32<0x128>(v);
  float o = v = sum_xor16(v);
  swap_halves(v, o);
  return v + o;
}
// v of the lane CTRL names, 0 where there is none (rows outside the row mask ROWS included)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t lanes_below(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xF, false));
}
// inclusive sum over this lane and the lower ones
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += lanes_below<0x111, 0xF>(v);   // row_shr:1
  v += lanes_below<0x112, 0xF>(v);
  v += lanes_below<0x114, 0xF>(v);
  v += lanes_below<0x118, 0xF>(v);
  v += lanes_below<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += lanes_below<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}
// sums over the wavefront's halves, in lanes 31 and 63
__device__ __forceinline__ uint32_t row_pair_sum(uint32_t v) {
  v += lanes_below<0x111, 0xF>(v);
  v += lanes_below<0x112, 0xF>(v);
  v += lanes_below<0x114, 0xF>(v);
  v += lanes_below<0x118, 0xF>(v);
  return v + lanes_below<0x142, 0xA>(v);
}
// maximum of numbers >= 0 (NaN is ignored), in every lane
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, 0.f);
  v = fmaxf(v, __uint_as_float(lanes_below<0x111, 0xF>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(lanes_below<0x112, 0xF>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(lanes_below<0x114, 0xF>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(lanes_below<0x118, 0xF>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(lanes_below<0x142, 0xA>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(lanes_below<0x143, 0xC>(__float_as_uint(v))));
  return __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(__float_as_uint(v)), 63)));
}

}  // namespace rdkv
