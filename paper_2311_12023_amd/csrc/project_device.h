// The last part of T = X L1, which is done by a launch of its own or beside another one.
#pragma once
#include "kernels.h"
#include "mfma_device.h"

namespace lq {

constexpr int XP_COLS = 64;          // columns of a partial tile of T

// hi = bf16(v), lo = bf16(v - hi): v = hi + lo + O(2^-17 v).
__device__ __forceinline__ void xp_split(floatx4 v, bf16x4& hi, bf16x4& lo) {
  hi = __builtin_convertvector(v, bf16x4);
  lo = __builtin_convertvector(v - __builtin_convertvector(hi, floatx4), bf16x4);
}

// T = sum of the partial tiles in range order, written as bf16 planes of rows_pad x Kd (the first Kd of the 64 columns): four
// columns at a time, items first, first + stride, ..
__device__ __forceinline__ void project_sum(const ProjectSum& t, int64_t first, int64_t step) {
  const int64_t q = t.Kd >> 2, total = t.rows_pad * q, stride = t.rows_pad * XP_COLS;
  for (int64_t i = first; i < total; i += step) {
    const int64_t row = i / q, c4 = (i % q) << 2;
    const float* p = t.part + row * XP_COLS + c4;
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < t.splits; s0 += 8) {     // the loads issued eight at a time
      floatx4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[u] = s0 + u < t.splits ? *reinterpret_cast<const floatx4*>(p + (int64_t)(s0 + u) * stride) : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += v[u];
    }
    bf16x4 hi, lo;
    xp_split(sum, hi, lo);
    *reinterpret_cast<bf16x4*>(t.th + row * t.Kd + c4) = hi;
    *reinterpret_cast<bf16x4*>(t.tl + row * t.Kd + c4) = lo;
  }
}

}  // namespace lq
