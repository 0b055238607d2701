// Device-side building blocks of the NF quantizer (Sections 2.2 and 3.2), shared by the stand-alone
// quantize / dequantize kernels and by the fused kernels of the decomposition loop.
//
// All arithmetic that decides a code or a scale index is written as single correctly rounded fp32
// operations (the library is compiled with -ffp-contract=off), so results are reproducible bit for bit:
//   normalised weight  fl32(u * fl32(1/s))           code = #{i : x >= thr[i]}
//   sigma = fl32(v / levels)   index = clamp(rne(fl32(s / sigma)), 0, levels)   s^ = fl32(index * sigma)
#pragma once

#include <hip/hip_fp16.h>

#include "lq_internal.h"

namespace lq {

typedef NfTables DevTables;
// Device address of the tables on the current device (uploads them on first use).
int device_tables(const DevTables** out);

template <int BITS>
struct Slot;
template <> struct Slot<2> { static constexpr int value = 0; };
template <> struct Slot<3> { static constexpr int value = 1; };
template <> struct Slot<4> { static constexpr int value = 2; };
template <> struct Slot<8> { static constexpr int value = 3; };

// LDS copy of one bit width's tables.
struct LdsTables {
  float code[256];
  float thr[260];
  uint8_t lut[512];
};

// Copies the tables of one bit width (slot) into LDS.  The caller places a barrier before the first use.
__device__ inline void load_tables_slot_nosync(const DevTables* __restrict__ tab, int slot, LdsTables& t) {
  for (int i = threadIdx.x; i < 256; i += blockDim.x) t.code[i] = tab->code[slot][i];
  for (int i = threadIdx.x; i < 260; i += blockDim.x) t.thr[i] = tab->thr[slot][i];
  for (int i = threadIdx.x; i < 128; i += blockDim.x)
    reinterpret_cast<uint32_t*>(t.lut)[i] = reinterpret_cast<const uint32_t*>(tab->lut[slot])[i];
}
__device__ inline void load_tables_slot(const DevTables* __restrict__ tab, int slot, LdsTables& t) {
  load_tables_slot_nosync(tab, slot, t);
  __syncthreads();
}

// The part of them that the bucket search reads.
template <int BITS>
__device__ inline void load_search_tables(const DevTables* __restrict__ tab, LdsTables& t) {
  constexpr int slot = Slot<BITS>::value;
  for (int i = threadIdx.x; i < (1 << BITS) + 2; i += blockDim.x) t.thr[i] = tab->thr[slot][i];
  for (int i = threadIdx.x; i < 128; i += blockDim.x)
    reinterpret_cast<uint32_t*>(t.lut)[i] = reinterpret_cast<const uint32_t*>(tab->lut[slot])[i];
  __syncthreads();
}

// Nearest code with ties to the lower index = number of thresholds <= x.
// 2 and 3 bits: the thresholds live in registers and are counted.  4 and 8 bits: a 512-bucket table in LDS
// gives the count of thresholds safely below x's bucket; at most two thresholds (8 bits) or one (4 bits, whose
// thresholds are more than twenty buckets apart) remain to be compared.  NaN compares false everywhere and lands
// on code 0 either way.
template <int BITS>
struct Thresholds {
  float r[(1 << BITS) - 1];
  __device__ Thresholds(const LdsTables&, const DevTables* __restrict__ tab) {      // uniform: scalar loads
#pragma unroll
    for (int i = 0; i < (1 << BITS) - 1; ++i) r[i] = tab->thr[Slot<BITS>::value][i];
  }
  __device__ inline uint32_t nearest(float x) const {
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < (1 << BITS) - 1; ++i) c += (x >= r[i]) ? 1u : 0u;
    return c;
  }
};
template <int COMPARES>
struct BucketSearch {
  const LdsTables& t;
  __device__ explicit BucketSearch(const LdsTables& tt) : t(tt) {}
  __device__ inline uint32_t nearest(float x) const {
    int j = (int)fmaf(x, 256.0f, 256.0f);
    j = j < 0 ? 0 : (j > 511 ? 511 : j);
    const uint32_t c0 = t.lut[j];
    uint32_t c = c0 + ((x >= t.thr[c0]) ? 1u : 0u);
    if constexpr (COMPARES == 2) c += (x >= t.thr[c0 + 1]) ? 1u : 0u;
    return c;
  }
};
template <> struct Thresholds<4> : BucketSearch<1> { __device__ Thresholds(const LdsTables& tt, const DevTables*) : BucketSearch<1>(tt) {} };
template <> struct Thresholds<8> : BucketSearch<2> { __device__ Thresholds(const LdsTables& tt, const DevTables*) : BucketSearch<2>(tt) {} };

// Code search of the decomposition's quantize pass: 16 buckets per unit, for 8 bits 256, and one comparison per weight.  The
// entry of x is found by one fused product whose sum keeps the bucket number in the mantissa bits from the third on, so that a mask
// leaves the entry's byte offset.  The sum
// rounds to 1/8 of a bucket: entry j serves x from (j - 1/16) / buckets - 1 to the same of j + 1, ends included, and counts the
// thresholds up to its lower end.  Thresholds are 1.27 (8 bits), 1.29 (4), 2.7 and 8 buckets apart at the least, so one at most is left
// to compare.  |x| is at most 1 + 2^-20 (a weight by the reciprocal of its block's largest one, or by 0), which is the last entry
// but one; NaN, whose mantissa may hold anything, becomes -1 first and takes code 0 (one instruction more per weight, 36 cells of
// 4096^2 31.3 ms with and without).  Up to 4 bits the 34 entries of 8 bytes lie
// in different LDS banks but for two pairs: with 256 buckets per unit for every width the quantize pass spent half of its LDS
// cycles on bank conflicts.
template <int BITS>
__host__ __device__ __forceinline__ uint32_t search_offset(float x) {
  constexpr float scale = (float)search_buckets(BITS), base = (float)(1 << 20) + scale;
  return __builtin_bit_cast(uint32_t, fmaf(x, scale, base)) & ((4u * search_buckets(BITS) - 1u) << 3);
}
template <int BITS>
__host__ __device__ __forceinline__ uint32_t search_code(const SearchEntry* table, float x) {
  x = fmaxf(x, -1.0f);
  const SearchEntry e = *reinterpret_cast<const SearchEntry*>(reinterpret_cast<const char*>(table) + search_offset<BITS>(x));
  return e.below + ((x >= e.thr) ? 1u : 0u);
}

// ---- cross-lane moves by DPP: quad_perm inside a quad of lanes; where every quad is uniform the mirror of a half row swaps the
// two quads of an 8-lane group and the mirror of a row the two halves of a 16-lane group ----
constexpr int DPP_QUAD_XOR1 = 0xB1, DPP_QUAD_XOR2 = 0x4E, DPP_ROW_HALF_MIRROR = 0x141, DPP_ROW_MIRROR = 0x140;
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
}

__device__ inline float run_absmax(const float (&t)[16]) {
  float m = 0.0f;
#pragma unroll
  for (int j = 0; j < 16; ++j) m = fmaxf(m, fabsf(t[j]));
  return m;
}

// fl32(1/s); 0 for an all-zero block or when the reciprocal overflows.
__device__ inline float safe_reciprocal(float s) {
  float r = 0.0f;
  if (s > 0.0f) {
    r = 1.0f / s;
    if (isinf(r)) r = 0.0f;
  }
  return r;
}

// ---- packed code stream: code j of run `run` occupies bits [(16*run + j)*BITS, +BITS) ------------
template <int BITS>
__device__ inline void store_codes(uint8_t* __restrict__ codes, int64_t run, const uint32_t (&c)[16]) {
  if constexpr (BITS == 8) {
    uint4 w;
    w.x = c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24);
    w.y = c[4] | (c[5] << 8) | (c[6] << 16) | (c[7] << 24);
    w.z = c[8] | (c[9] << 8) | (c[10] << 16) | (c[11] << 24);
    w.w = c[12] | (c[13] << 8) | (c[14] << 16) | (c[15] << 24);
    *reinterpret_cast<uint4*>(codes + run * 16) = w;
  } else {
    uint64_t w = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) w |= (uint64_t)c[j] << (j * BITS);
    if constexpr (BITS == 4) {
      *reinterpret_cast<uint2*>(codes + run * 8) = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
    } else if constexpr (BITS == 2) {
      *reinterpret_cast<uint32_t*>(codes + run * 4) = (uint32_t)w;
    } else {   // 3 bits: 48 bits, 2-byte aligned
      uint16_t* p = reinterpret_cast<uint16_t*>(codes + run * 6);
      p[0] = (uint16_t)w; p[1] = (uint16_t)(w >> 16); p[2] = (uint16_t)(w >> 32);
    }
  }
}

template <int BITS>
__device__ inline void load_codes(const uint8_t* __restrict__ codes, int64_t run, uint32_t (&c)[16]) {
  if constexpr (BITS == 8) {
    const uint4 w = *reinterpret_cast<const uint4*>(codes + run * 16);
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < 16; ++j) c[j] = (ww[j >> 2] >> ((j & 3) * 8)) & 0xffu;
  } else {
    uint64_t w;
    if constexpr (BITS == 4) {
      const uint2 u = *reinterpret_cast<const uint2*>(codes + run * 8);
      w = (uint64_t)u.x | ((uint64_t)u.y << 32);
    } else if constexpr (BITS == 2) {
      w = *reinterpret_cast<const uint32_t*>(codes + run * 4);
    } else {
      const uint16_t* p = reinterpret_cast<const uint16_t*>(codes + run * 6);
      w = (uint64_t)p[0] | ((uint64_t)p[1] << 16) | ((uint64_t)p[2] << 32);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) c[j] = (uint32_t)(w >> (j * BITS)) & ((1u << BITS) - 1u);
  }
}

// ---- quad layout: one lane holds 4 consecutive weights, 4 lanes a 16-weight run, so that every wavefront
// load / store covers one contiguous stretch.  Codes of quad `quad` occupy bits [quad*4*BITS, +4*BITS).
template <int BITS>
__device__ inline void load_quad_codes(const uint8_t* __restrict__ codes, int64_t quad, uint32_t (&c)[4]) {
  uint32_t w;
  if constexpr (BITS == 8) w = *reinterpret_cast<const uint32_t*>(codes + quad * 4);
  else if constexpr (BITS == 4) w = *reinterpret_cast<const uint16_t*>(codes + quad * 2);
  else if constexpr (BITS == 2) w = codes[quad];
  else {   // 3 bits: 12 bits starting at bit 12*quad = byte floor(1.5*quad), nibble-aligned
    const int64_t byte = (quad * 3) >> 1;
    w = ((uint32_t)codes[byte] | ((uint32_t)codes[byte + 1] << 8)) >> ((quad & 1) * 4);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = (w >> (j * BITS)) & ((1u << BITS) - 1u);
}

// ---- second-level (integer) scale quantization -------------------------------------------------
// Maximum over the `width` (power of two, <= 64, aligned) consecutive lanes of a wavefront: DPP moves up to 16 lanes
// (quad permutes, then half-row and row mirrors, which act as xor 4 and xor 8 on quad-uniform values), the LDS
// crossbar beyond.  `width` is uniform, so the branches are too.
__device__ __forceinline__ float lanes_max(float x, int width) {
  if (width > 1) x = fmaxf(x, dpp_move<DPP_QUAD_XOR1>(x));
  if (width > 2) x = fmaxf(x, dpp_move<DPP_QUAD_XOR2>(x));
  if (width > 4) x = fmaxf(x, dpp_move<DPP_ROW_HALF_MIRROR>(x));
  if (width > 8) x = fmaxf(x, dpp_move<DPP_ROW_MIRROR>(x));
  if (width > 16) x = fmaxf(x, __shfl_xor(x, 16));
  if (width > 32) x = fmaxf(x, __shfl_xor(x, 32));
  return x;
}

// Maximum over the `width` consecutive lanes (power of two, 16 .. the workgroup's size, aligned) that hold one scale
// group.  s_wave: one float of LDS per wavefront.  Contains barriers when
// width > 64, so every thread of the workgroup must call it.
__device__ inline float group_max(float x, int width, float* s_wave) {
  x = lanes_max(x, width < 64 ? width : 64);
  if (width > 64) {
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) s_wave[wave] = x;
    __syncthreads();
    const int per = width >> 6;             // waves per group, a power of two
    const int base = wave & ~(per - 1);
    float m = s_wave[base];
    for (int i = 1; i < per; ++i) m = fmaxf(m, s_wave[base + i]);
    x = m;
    __syncthreads();
  }
  return x;
}

__device__ inline uint32_t scale_index(float s, float sigma, int levels) {
  if (!(sigma > 0.0f)) return 0u;
  float r = rintf(s / sigma);
  r = fminf(fmaxf(r, 0.0f), (float)levels);
  return (uint32_t)r;
}

__device__ inline float block_scale(uint32_t idx, float v_stored, int levels) {
  const float sigma = v_stored / (float)levels;
  return (float)idx * sigma;
}

// v / levels with inv = fl32(1 / levels), without a division: the quotient by the reciprocal, corrected by its remainder,
// which the fused product leaves exact (Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", 1990).  Equal to the division for every v >= 0 and every `levels` that a configuration can have (all 2^31
// bit patterns compared on the host).  The maximum is for v = infinity, where the remainder is inf - inf: what is added
// to the infinite quotient then only has to be a number.
__host__ __device__ inline float sigma_by_reciprocal(float v, float levels, float inv) {
  const float q = v * inv;
  return fmaf(fmaxf(fmaf(-q, levels, v), -3.402823466e38f), inv, q);
}
// block_scale for kernels whose inner loop it is in.
__device__ __forceinline__ float block_scale_by_reciprocal(uint32_t idx, float v_stored, int levels, float inv) {
  return (float)idx * sigma_by_reciprocal(v_stored, (float)levels, inv);
}

// cast(v, b2): round to nearest even into the storage type, returned as fp32.
__device__ inline float cast_group_scale(float v, int v_dtype) {
  if (v_dtype == LQ_V_BF16) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7f800000u) != 0x7f800000u) {
      u += 0x7fffu + ((u >> 16) & 1u);
      u &= 0xffff0000u;
    }
    return __uint_as_float(u);
  }
  if (v_dtype == LQ_V_FP16) return __half2float(__float2half_rn(v));
  return v;
}

}  // namespace lq
