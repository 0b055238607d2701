// Vector types and operand conversions that the kernels of the large products share.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lq {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));   // native vector: arrays of it stay in registers
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));

// a = hi + lo + O(2^-17 a) with hi, lo in bf16.
__device__ __forceinline__ void split_bf16(floatx2 v, bf16x2& hi, bf16x2& lo) {
  hi = __builtin_convertvector(v, bf16x2);
  const floatx2 back = __builtin_convertvector(hi, floatx2);
  lo = __builtin_convertvector(v - back, bf16x2);
}

// Operand layout of a wide matrix for column_gemm_kernel: [k / 32][row / 16][hi, lo][lane] of 16 bytes; lane 16 q + n holds row
// n, k = 4 q + 0..3 and 16 + 4 q + 0..3.  Stores four values of one row; k is a multiple of four, row_tiles = rows / 16.
__device__ __forceinline__ void store_packed(uintx2* packed, int row_tiles, int row, int64_t k, floatx4 v) {
  bf16x2 h0, l0, h1, l1;
  split_bf16(floatx2{v[0], v[1]}, h0, l0);
  split_bf16(floatx2{v[2], v[3]}, h1, l1);
  const int kk = (int)(k & 31), lane = 16 * ((kk & 15) >> 2) + (row & 15);
  uintx2* o = packed + (((size_t)(k >> 5) * row_tiles + (row >> 4)) * 2 * 64 + lane) * 2 + (kk >> 4);
  o[0] = __builtin_bit_cast(uintx2, bf16x4{h0[0], h0[1], h1[0], h1[1]});
  o[128] = __builtin_bit_cast(uintx2, bf16x4{l0[0], l0[1], l1[0], l1[1]});
}

// The lo plane of the residual: one byte per element, the upper byte of the fp16 number 2^11 (a - hi) (sign, five exponent
// bits, two fraction bits).
constexpr float LO8_SCALE = 2048.0f;

// Power of two xs with |x| xs <= 2^13 for the rows of a wide matrix whose largest squared row norm is lam0.
__device__ __forceinline__ float x_scale_from(double lam0) {
  const float s = (float)lam0;
  if (!(s > 0.0f) || !(s < 3.0e38f)) return 1.0f;
  return exp2f(13.0f - ceilf(0.5f * log2f(s)));
}

}  // namespace lq
