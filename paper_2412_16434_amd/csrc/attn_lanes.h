// What the attention kernels share: operand layouts of the 32x32x16 bf16 matrix instruction, exchanges between lanes.
#pragma once

#include "common.h"

namespace symph {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Row r (0..31) of the A operand of S^T = K Q^T holds key key_of_row(r) of the 32-key block, chosen so that the
// MFMA result registers 8*u .. 8*u+7 of a lane in half-wave g2 are keys 16*u + 8*g2 + 0..7.
__device__ __forceinline__ int key_of_row(int r) {
  const int j = r & 3, gg = (r >> 2) & 1, i = r >> 3;
  return 16 * (i >> 1) + 8 * gg + 4 * (i & 1) + j;
}

// ds_read_b64_tr_b16: the 16 lanes of a group hand in the addresses of a 4 x 16 tile of 16-bit values (lanes
// 4e .. 4e+3 cover row e, 4 values each) and lane i gets column i, i.e. 4 consecutive rows of one column.
__device__ __forceinline__ s16x4 lds_read_tr16(const __bf16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(const_cast<__bf16*>(p)));
}

// Lanes l and l^32 hold the two halves of one query's keys.  v_permlane32_swap_b32 a, b exchanges lanes 32..63 of a
// with lanes 0..31 of b, so starting from two copies of x it leaves a = low half twice, b = high half twice.
// Written as inline assembly: with this compiler the builtin hands back the first register for both results.
__device__ __forceinline__ void swap_halves(float x, float& lo_twice, float& hi_twice) {
  float a = x, b = x;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));  // a pure function of a, b: free to be scheduled
  lo_twice = a;
  hi_twice = b;
}
__device__ __forceinline__ float max_across_halves(float x) {
  float lo, hi;
  swap_halves(x, lo, hi);
  return fmaxf(lo, hi);
}
__device__ __forceinline__ float sum_across_halves(float x) {
  float lo, hi;
  swap_halves(x, lo, hi);
  return lo + hi;
}

}  // namespace symph
