// Forward product with a decomposed weight for 9 to 128 rows of X (decoding many sequences at once, short prompts):
// Y[m x N] = X dequant(codes) + (X L1) L2.  Two launches: the kernel below multiplies X with [Q | L1]
// over ranges of the reduction, qmatvec_finish_kernel or rows_finish_kernel adds the ranges and the product (X L1) L2.
//
// A lane fetches half a 16-weight run of eight reduction rows, turns them straight into the operand layout of
// v_mfma_f32_16x16x32_bf16 (8 column sets of 16 columns) and multiplies them with rows of X that it splits into bf16
// halves on the way; only the sums are staged.  A workgroup owns 128 columns at a time; its eight wavefronts take
// turns at the 32-deep reduction steps and their sums are added in order through LDS.  Every weight is turned into operands for at
// most 48 rows, so that takes the time, not the products, and there are two forms of it:
// - Blocks of 64 weights and more, where scales_in_x_ahead and scaled_rounds say so.  The 64 or 128 columns of a row that a tile has in
//   a block share one scale, so X Q is the product of X, its columns times these scales, with values of the code book, whose bf16
//   halves come from a table for two rows of Q at a time (QrTable).  A wavefront computes a step's scales one per lane and hands them
//   out through LDS.  X times the scale goes in as three bf16 (precision 1: two): five products (two).
// - Otherwise: extract, look up, scale and split every weight into two bf16 (one): three
//   products (one).
// Per wavefront and step of 4096 x 11008 at 24 rows the loop has 349 vector instructions in the first form and 490 in the second; what
// is left is latency: two wavefronts per SIMD, loads one step ahead, and the first fetch (behind the first segment: asked for with
// that one's last step) and last sum of each workgroup.  scales_in_x_ahead has both sides' times.  With two parts of X times the scale
// (four products) 24 rows took 26.2 us instead of 28.5, but rows of X that are exact in bf16, which the second form does not round,
// came out with an error of 3.2e-6 instead of 2.5e-6 (precision 1: 1.9e-3 instead of 1.7e-3); now 0.7e-6 (4 bits), 1.7e-6 (8) and
// 1.1e-3, 1.2e-3, and for any fp32 X the same instead of 4.4e-6 and 2.3e-3.  (X times the scale below 2^-112 loses bits: 1e-5 where
// results are 1e-34.)  What did not help: a wavefront per 64 columns and four per step, two steps in flight (twice the loads of X: 29 us
// at 24 rows, 42 at 48, against 27 and 37 then), one copy of the table (bank conflicts: 29.4).
// Second form, whole call on 4096 x 11008, NF4, rank 64 (4096 x 4096): 24 rows 79 -> 32 us (45 -> 20), 64 rows 84 -> 50 us (47 -> 27),
// 128 rows 94 -> 85 us (52 -> 42) against the kernel for large m, whose steps take 2 us whatever they multiply (256-row tiles
// of X staged through LDS, a barrier per step).  At 192 rows that kernel is ahead on the wide matrix (95 against 111 us)
// and level on the square one, so the line is drawn at 128; rows_kernel_ahead in lq_api_matmul.cpp has the large weights
// on which it is ahead from 65 or 97 rows on.  What did not help: 256 columns per workgroup (twice the
// accumulators, half the wavefronts in flight: 37 us at 24 rows), four wavefronts per SIMD (registers spill: 80 us).
#include <algorithm>

#include "dense_device.h"
#include "kernels.h"
#include "nf_device.h"
#include "profiler.h"

namespace lq {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int QR_SETS = 8;           // columns per lane
constexpr int QR_COLS = 16 * QR_SETS;   // columns of Q per workgroup
constexpr int QR_DCOLS = 64;         // columns of L1 per workgroup
constexpr int QR_WAVES = 8;
constexpr int QR_TILES = 3;          // 16-row tiles of X per workgroup at most (four spill registers)
struct QrArgs {
  const float* X; int64_t ldx;
  const uint8_t* codes; const uint8_t* sidx; const float* v;
  const float* D; int64_t ldd; int Nd;       // L1: K x Nd
  int d_vec;                                 // its rows can be read as float4
  float* part;                               // segment z of a tile, row i of X Q at part + (z * m + i) * N
  float* tpart;                              // segment z of a tile, row i of X L1 at tpart + (z * m + i) * Nd
  int64_t K, N;
  int m, ksteps, steps, total, per_wg, tiles_q;   // steps of a tile: with work, counted; counted in all tiles, per workgroup
  int block_shift, group_shift, levels;
  float inv_levels;
  const DevTables* tables;
};

__device__ __forceinline__ void split_pair(float a, float b, bf16x2& hi, bf16x2& lo) {
  const floatx2 v = {a, b};
  hi = __builtin_convertvector(v, bf16x2);
  lo = __builtin_convertvector(v - __builtin_convertvector(hi, floatx2), bf16x2);
}
template <bool SPLIT>
__device__ __forceinline__ void split8(const float (&w)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    bf16x2 h, l;
    if constexpr (SPLIT) split_pair(w[i], w[i + 1], h, l);
    else { h = __builtin_convertvector(floatx2{w[i], w[i + 1]}, bf16x2); l = h; }
    hi[i] = h[0]; hi[i + 1] = h[1];
    if constexpr (SPLIT) { lo[i] = l[0]; lo[i + 1] = l[1]; }
  }
}

// w as the sum of N bf16 parts, largest first: what they leave is about 2^-9 of the one before the last, each.
template <int N>
__device__ __forceinline__ void split_parts(const float (&w)[8], bf16x8 (&part)[N]) {
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    floatx2 v = {w[i], w[i + 1]};
#pragma unroll
    for (int p = 0; p < N; ++p) {
      const bf16x2 b = __builtin_convertvector(v, bf16x2);
      part[p][i] = b[0]; part[p][i + 1] = b[1];
      if (p + 1 < N) v -= __builtin_convertvector(b, floatx2);
    }
  }
}

// Codes of half a 16-weight run (8 weights, `half` its position) as they come from memory.
template <int BITS>
struct HalfRun { uint32_t w[BITS == 8 ? 2 : 1]; };
template <int BITS>
__device__ __forceinline__ HalfRun<BITS> load_half(const uint8_t* run, uint32_t half) {
  HalfRun<BITS> r;
  if constexpr (BITS == 8) {
    const uint2 t = *reinterpret_cast<const uint2*>(run + 8 * half);
    r.w[0] = t.x; r.w[1] = t.y;
  } else if constexpr (BITS == 4) {
    r.w[0] = *reinterpret_cast<const uint32_t*>(run + 4 * half);
  } else if constexpr (BITS == 2) {
    r.w[0] = *reinterpret_cast<const uint16_t*>(run + 2 * half);
  } else {                                   // bytes 3 half .. 3 half + 2 of six are bytes half .. half + 2 of these, 2-byte aligned
    __builtin_memcpy(r.w, run + 2 * half, 4);
  }
  return r;
}
// Byte offset of code J's value in the table (4 times the code).  4 bits: the codes are first moved into bytes, four at a
// time, so that a code costs one more instruction instead of a shift and a mask.
template <int BITS>
__device__ __forceinline__ uint2 spread_half(const HalfRun<BITS>& r, uint32_t half) {
  if constexpr (BITS == 8) return make_uint2(r.w[0], r.w[1]);
  else if constexpr (BITS == 4) return make_uint2((r.w[0] << 2) & 0x3c3c3c3cu, (r.w[0] >> 2) & 0x3c3c3c3cu);   // even, odd codes
  else if constexpr (BITS == 3) return make_uint2((r.w[0] >> (8 * half)) << 2, 0u);
  else return make_uint2(r.w[0] << 2, 0u);
}
template <int BITS, int J>
__device__ __forceinline__ uint32_t code_offset(uint2 r) {
  if constexpr (BITS == 8) return __builtin_amdgcn_ubfe(J < 4 ? r.x : r.y, 8 * (J % 4), 8) << 2;
  else if constexpr (BITS == 4) return __builtin_amdgcn_ubfe(J % 2 ? r.y : r.x, 8 * (J / 2), 8);
  else return (r.x >> (J * BITS)) & (((1u << BITS) - 1u) << 2);
}

// The table of the form with the scales in X: for codes of up to 4 bits, for every pair of them, a word of their bf16 high halves
// (the first one's in the lower half) 32 times and a word of their low halves 32 times, for 8 bits a word of both halves of every
// code 32 times: a lane reads its own copy, and no two of the 32 lanes that LDS serves at a time meet in a bank (a single copy of
// the 256 pairs of 4-bit codes took 60 % of the reads' cycles for conflicts).
template <int BITS> struct QrTable {
  static constexpr int entries = BITS == 8 ? 256 : 1 << (2 * BITS), shift = BITS == 8 ? 7 : 8, words = entries << (shift - 2);
};
// Codes of this lane in one row: with NBLK = 1 columns 8 c + j in set j, with NBLK = 2 columns 4 c + j of the first 64 and then of the
// second.  They stay as they come from memory until words() puts set j at bits [j BITS, + BITS): put together at once they would
// be waited for at once.
template <int BITS, int NBLK>
struct RowCodes {
  uint32_t lo, hi;
  // byte offset of the lane's first code in a row
  __device__ __forceinline__ static uint32_t lane_offset(int c) {
    if constexpr (NBLK == 2) return (uint32_t)(4 * BITS * c) / 8u;
    else return BITS == 3 ? (uint32_t)(c >> 1) * 6u + 2u * (c & 1) : (uint32_t)(BITS * c);
  }
  // `row` (of codes, uniform) + `lane`; `second`: bytes to the second 64 columns (uniform)
  __device__ __forceinline__ void load(const uint8_t* row, uint32_t lane, uint32_t second) {
    if constexpr (BITS == 8) {
      lo = *reinterpret_cast<const uint32_t*>(row + lane);
      hi = *reinterpret_cast<const uint32_t*>(row + (NBLK == 2 ? second : 4u) + lane);
    } else if constexpr (BITS == 3 && NBLK == 1) {        // 2-byte aligned
      hi = 0;
      __builtin_memcpy(&lo, row + lane, 4);
    } else if constexpr (BITS == 3) {        // the 12 bits from bit 12 c on
      uint16_t w[2];
      __builtin_memcpy(w, row + lane, 2);
      __builtin_memcpy(w + 1, row + second + lane, 2);
      lo = w[0]; hi = w[1];
    } else if constexpr (NBLK == 1) {
      hi = 0;
      if constexpr (BITS == 4) lo = *reinterpret_cast<const uint32_t*>(row + lane);
      else lo = *reinterpret_cast<const uint16_t*>(row + lane);
    } else if constexpr (BITS == 4) {
      lo = *reinterpret_cast<const uint16_t*>(row + lane);
      hi = *reinterpret_cast<const uint16_t*>(row + second + lane);
    } else {
      lo = (row + lane)[0]; hi = (row + second + lane)[0];
    }
  }
  // What is done with a step's codes is not done before this: at the end of the step before, they would be waited for.
  __device__ __forceinline__ void arrived() {
    asm("" : "+v"(lo));
    if constexpr (BITS == 8 || NBLK == 2) asm("" : "+v"(hi));
  }
  __device__ __forceinline__ void words(int c, uint32_t (&w)[2]) const {
    w[0] = lo; w[1] = hi;
    if constexpr (BITS == 3 && NBLK == 1) w[0] = lo >> (8 * (c & 1));
    else if constexpr (BITS == 3) {
      const uint32_t sh = 4 * (c & 1);
      w[0] = ((lo >> sh) & 0xfffu) | (((hi >> sh) & 0xfffu) << 12);
    } else if constexpr (BITS != 8 && NBLK == 2) w[0] = lo | (hi << (4 * BITS));
  }
};

// Four columns from `col` (a multiple of 4) of row `row` of X times rows k0 .. k1 - 1 of Q, one element at a time; NaN at once where
// X holds one.
template <int BITS>
__device__ __forceinline__ floatx4 plain_sum(const QrArgs& a, int row, int64_t col, int64_t k0, int64_t k1) {
  const float* x = a.X + (int64_t)row * a.ldx;
  bool nan = false;
#pragma unroll 8
  for (int64_t k = k0; k < k1; k += 4) {
    const floatx4 v = *reinterpret_cast<const floatx4*>(x + k);
    nan = nan || isnan(v[0]) || isnan(v[1]) || isnan(v[2]) || isnan(v[3]);
  }
  floatx4 o = {0.f, 0.f, 0.f, 0.f};
  if (nan) return o + NAN;
  const float* book = a.tables->code[Slot<BITS>::value];
  const int quad = (int)(col & 15) >> 2;                             // of the 16-weight run
#pragma unroll 1
  for (int64_t k = k0; k < k1; ++k) {
    const uint8_t* from = a.codes + (uint64_t)((k * a.N + col) >> 4) * (2 * BITS) + ((4 * BITS * quad) >> 3);
    uint32_t w = from[0];
    if constexpr (BITS > 2) w |= (uint32_t)from[1] << 8;
    if constexpr (BITS == 8) w |= (uint32_t)from[2] << 16 | (uint32_t)from[3] << 24;
    if constexpr (BITS == 3) w >>= 4 * (quad & 1);
    const uint32_t blk = (uint32_t)((k * a.N + col) >> a.block_shift);
    const float scale = block_scale_by_reciprocal(a.sidx[blk], a.v[blk >> a.group_shift], a.levels, a.inv_levels);
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = fmaf(x[k], book[__builtin_amdgcn_ubfe(w, BITS * j, BITS)] * scale, o[j]);
  }
  return o;
}

// The steps of all column tiles, in order (tile, step), are dealt out in equal contiguous shares, so that every compute unit
// gets the same work whatever the number of tiles; a workgroup's part of a tile is one segment, numbered within the tile.
// NBLK: 0 the form for small blocks, else the number of blocks of a tile's 128 columns.
template <int BITS, int RT, bool SPLIT, int NBLK>
__global__ __launch_bounds__(64 * QR_WAVES, 2) void qrows_kernel(QrArgs a) {
  constexpr int TABLE = NBLK == 0 ? 1 << BITS : QrTable<BITS>::words;
  typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
  __shared__ struct {
    uint32_t code[TABLE];                    // first: a code's offset in the table is its LDS address
    __attribute__((aligned(16))) float scale[NBLK == 0 ? 4 : QR_WAVES * NBLK * 32];
    __attribute__((aligned(16))) float sum[QR_WAVES][4][QR_SETS][64];
  } sh;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int c = lane & 15, q = lane >> 4;
  const int row0 = (int)blockIdx.y * (16 * RT);
  const int wg = (int)blockIdx.x;
  const int end = (wg + 1) * a.per_wg < a.total ? (wg + 1) * a.per_wg : a.total;

  // rows of X that this lane feeds to the MFMAs (past the last one: computed and never stored)
  const float* xrow[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    int r = row0 + 16 * t + c;
    r = r < a.m ? r : a.m - 1;
    xrow[t] = a.X + (int64_t)r * a.ldx + 8 * q;
  }
  floatx4 xv[RT][2];
  auto fetch_x = [&](int s) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      xv[t][0] = *reinterpret_cast<const floatx4*>(xrow[t] + 32 * (int64_t)s);
      xv[t][1] = *reinterpret_cast<const floatx4*>(xrow[t] + 32 * (int64_t)s + 4);
    }
  };
  bf16x8 xh[RT], xl[RT];
  auto split_x = [&]() {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const float x[8] = {xv[t][0][0], xv[t][0][1], xv[t][0][2], xv[t][0][3], xv[t][1][0], xv[t][1][1], xv[t][1][2], xv[t][1][3]};
      split8<SPLIT>(x, xh[t], xl[t]);
    }
  };
  floatx4 acc[RT][QR_SETS];
  auto multiply = [&](const float (&w)[8], auto set) __attribute__((always_inline)) {
    constexpr int j = decltype(set)::value;
    bf16x8 wh, wl;
    split8<SPLIT>(w, wh, wl);
    if constexpr (SPLIT) {
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl[t], wh, acc[t][j], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh[t], wl, acc[t][j], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh[t], wh, acc[t][j], 0, 0, 0);
  };

  // The form with the scales in X: what a step needs of X, codes and scales, one step ahead and across segments.
  constexpr int NX = NBLK == 2 ? 2 : 1, XPARTS = SPLIT ? 3 : 2;
  // The code book times this is off by 5.0e-7 as a sum of two bf16, without it by 1.9e-6 (the other widths gain nothing by a factor).
  constexpr float gain = BITS == 4 && SPLIT ? 1.828125f : 1.0f;
  typedef RowCodes<BITS, NBLK == 0 ? 1 : NBLK> Row;
  const uint32_t run_bytes = (uint32_t)(a.N / 16 * (2 * BITS)), row_blocks = (uint32_t)(a.N >> a.block_shift);   // of a row
  const uint32_t row_lane = (uint32_t)(8 * q) * run_bytes + Row::lane_offset(c);
  const uint32_t lane4 = 4u * (lane & 31);                              // this lane's copy of a table entry
  float* const scales = sh.scale + (NBLK == 0 ? 0 : wave * (NX * 32));
  Row cw[8];
  uint32_t si = 0;
  float vv = 0.f;
  auto fetch_step = [&](int tile, int s) __attribute__((always_inline)) {
    const int64_t col0 = (int64_t)tile * QR_COLS;
    const bool two = NBLK == 2 && col0 + 64 < a.N;                      // N is a multiple of the block; else the first 64 columns again
    const uint32_t second = two ? 8u * BITS : 0u;
    uint64_t step = (uint64_t)(32 * (uint32_t)s) * run_bytes + (uint64_t)(col0 / 16) * (2 * BITS);
    asm("" : "+s"(step));                                               // one lane offset for all rows instead of a pointer each
#pragma unroll
    for (int i = 0; i < 8; ++i) cw[i].load(a.codes + step + (uint64_t)((uint32_t)i * run_bytes), row_lane, second);
    // one scale per lane: row lane % 32 of the step, block lane / 32
    const uint32_t blk = (32 * (uint32_t)s + (uint32_t)(lane & 31)) * row_blocks + (uint32_t)((col0 + (two && lane >= 32 ? 64 : 0)) >> a.block_shift);
    si = a.sidx[blk];
    vv = a.v[blk >> a.group_shift];
    fetch_x(s);
  };

  bool table = false, ready = false;
  for (int pos = wg * a.per_wg; pos < end;) {
    const int tile = pos / a.steps, s0 = pos - tile * a.steps;
    int s1 = a.steps - s0 < end - pos ? a.steps : s0 + (end - pos);
    // The steps of all tiles fit an int; in the form without scales in X the quotient of 32 bits changes how the compiler orders the
    // loop's reads of the code book (4 bits, precision 1, 48 rows x 4096 x 11008: 33.3 instead of 32.3 us).
    const int segment = wg - (NBLK == 0 ? (int)((int64_t)tile * a.steps / a.per_wg) : tile * a.steps / a.per_wg);
    pos += s1 - s0;
    s1 = s1 < a.ksteps ? s1 : a.ksteps;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int j = 0; j < QR_SETS; ++j) acc[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const bool dense = tile >= a.tiles_q;
    int s = s0 + wave;
    if (!dense && NBLK > 0) {
      if (!ready && s < s1) fetch_step(tile, s);
      ready = false;
      int next_s1 = 0;                         // steps of the next segment, if it is one of Q
      if (pos < end && tile + 1 < a.tiles_q) next_s1 = end - pos < a.ksteps ? end - pos : a.ksteps;
      if (!table) {
        const float* book = a.tables->code[Slot<BITS>::value];
#pragma unroll
        for (int i = 0; i < (QrTable<BITS>::words / 4 + 64 * QR_WAVES - 1) / (64 * QR_WAVES); ++i) {
          const int at = 16 * (tid + 64 * QR_WAVES * i), e = at >> QrTable<BITS>::shift;     // 16 bytes, entry
          bf16x2 hi, lo;
          uint32_t w;
          if constexpr (BITS == 8) {
            split_pair(book[e], 0.f, hi, lo);
            w = __builtin_bit_cast(uint32_t, bf16x2{hi[0], lo[0]});
          } else {
            const int pr = e < QrTable<BITS>::entries ? e : 0;
            split_pair(gain * book[pr & ((1 << BITS) - 1)], gain * book[pr >> BITS], hi, lo);
            w = __builtin_bit_cast(uint32_t, at & 128 ? lo : hi);
          }
          if (e < QrTable<BITS>::entries) *reinterpret_cast<uint4*>(reinterpret_cast<char*>(sh.code) + at) = make_uint4(w, w, w, w);
        }
        __syncthreads();
        table = true;
      }
      for (; s < s1; s += QR_WAVES) {
#pragma unroll
        for (int i = 0; i < 8; ++i) cw[i].arrived();
        asm("" : "+v"(si), "+v"(vv));
        if (NBLK == 2 || lane < 32) scales[lane] = block_scale_by_reciprocal(si, vv, a.levels, a.inv_levels) * (1.0f / gain);
        // fields of 2 BITS bits: the codes of rows 2 p and 2 p + 1 in set 2 f (pair[p][0]) and 2 f + 1 (pair[p][1])
        uint32_t pair[4][2];
        uint32_t codes[8][2];
#pragma unroll
        for (int i = 0; i < 8; ++i) cw[i].words(c, codes[i]);
        if constexpr (BITS != 8) {
          constexpr uint32_t M = BITS == 4 ? 0x0f0f0f0fu : BITS == 3 ? 07070707u : 0x3333u;
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const uint32_t u = codes[2 * p][0], d = codes[2 * p + 1][0];
            pair[p][0] = (u & M) | ((d << BITS) & ~M);
            pair[p][1] = ((u >> BITS) & M) | (d & ~M);
          }
        }
        __builtin_amdgcn_wave_barrier();
        float xs[NX][RT][8];
#pragma unroll
        for (int b = 0; b < NX; ++b) {
          const floatx4 sl = *reinterpret_cast<const floatx4*>(scales + 32 * b + 8 * q), su = *reinterpret_cast<const floatx4*>(scales + 32 * b + 8 * q + 4);
#pragma unroll
          for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) xs[b][t][e] = xv[t][e >> 2][e & 3] * (e < 4 ? sl[e & 3] : su[e & 3]);
        }
        // next: this tile's step, or the first one of the segment behind this one, or (nothing left) the same again
        int next_tile = tile, next = s;
        if (s + QR_WAVES < s1) next = s + QR_WAVES;
        else if (wave < next_s1) { next_tile = tile + 1; next = wave; ready = true; }
        fetch_step(next_tile, next);
        __builtin_amdgcn_sched_barrier(0);
        for_each_block<NX>([&](auto block) {
          constexpr int b = decltype(block)::value;
          // The values have one or two parts.  X times the scale has one more: rounding both sides alike would add an error that
          // rounding the scaled weight does not make where X is exact in bf16.
          if constexpr (b > 0) __builtin_amdgcn_sched_barrier(0);
          bf16x8 xp[RT][XPARTS];
#pragma unroll
          for (int t = 0; t < RT; ++t) split_parts(xs[b][t], xp[t]);
          constexpr int SETS = RT < 2 ? 2 : 1;           // sets at a time: successive products are independent of one another
          for_each_block<QR_SETS / NX / SETS>([&](auto set) {
            constexpr int j0 = QR_SETS / NX * b + SETS * decltype(set)::value;
            uintx4 h[SETS], l[SETS];
#pragma unroll
            for (int i = 0; i < SETS; ++i)
#pragma unroll
              for (int p = 0; p < 4; ++p) {
                const int j = j0 + i;
                const char* table = reinterpret_cast<const char*>(sh.code);
                if constexpr (BITS == 8) {
                  const uint32_t u = *reinterpret_cast<const uint32_t*>(table + ((__builtin_amdgcn_ubfe(codes[2 * p][j / 4], 8 * (j % 4), 8) << 7) | lane4));
                  const uint32_t d = *reinterpret_cast<const uint32_t*>(table + ((__builtin_amdgcn_ubfe(codes[2 * p + 1][j / 4], 8 * (j % 4), 8) << 7) | lane4));
                  h[i][p] = __builtin_amdgcn_perm(d, u, 0x05040100);
                  l[i][p] = __builtin_amdgcn_perm(d, u, 0x07060302);
                } else {
                  const uint32_t f = pair[p][j % 2];
                  const uint32_t at = BITS == 4 ? __builtin_amdgcn_perm(f, lane4, 0x0c0c0000u | ((4u + j / 2) << 8))
                                                : (__builtin_amdgcn_ubfe(f, 2 * BITS * (j / 2), 2 * BITS) << 8) | lane4;
                  h[i][p] = *reinterpret_cast<const uint32_t*>(table + at);
                  l[i][p] = SPLIT ? *reinterpret_cast<const uint32_t*>(table + at + 128) : 0u;
                }
              }
            auto product = [&](int part, const uintx4 (&w)[SETS]) __attribute__((always_inline)) {
#pragma unroll
              for (int i = 0; i < SETS; ++i)
#pragma unroll
                for (int t = 0; t < RT; ++t)
                  acc[t][j0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xp[t][part], __builtin_bit_cast(bf16x8, w[i]), acc[t][j0 + i], 0, 0, 0);
            };
            if constexpr (SPLIT) { product(2, h); product(1, l); product(0, l); }
            product(1, h);
            product(0, h);
          });
        });
        __builtin_amdgcn_wave_barrier();
      }
    } else if (!dense) {
      const int64_t col = (int64_t)tile * QR_COLS + QR_SETS * c;
      const int64_t colc = col < a.N ? col : 0;                       // N is a multiple of 16
      const uint32_t run_bytes = (uint32_t)(a.N / 16 * (2 * BITS));   // of a row
      const uint32_t row_blocks = (uint32_t)(a.N >> a.block_shift);
      const uint32_t half = (uint32_t)(colc / 8) & 1u;
      const uint32_t lane_codes = (uint32_t)(8 * q) * run_bytes + (uint32_t)(colc / 16 * (2 * BITS));
      const uint32_t lane_block = (uint32_t)(8 * q) * row_blocks + (uint32_t)(colc >> a.block_shift);
      HalfRun<BITS> cw[8];
      uint32_t si[8];
      float vv[8];
      auto fetch_w = [&](int s) {
        const uint8_t* base = a.codes + (uint64_t)(32 * (uint32_t)s) * run_bytes;
        const uint32_t blk0 = 32 * (uint32_t)s * row_blocks + lane_block;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          cw[i] = load_half<BITS>(base + (lane_codes + (uint32_t)i * run_bytes), half);
          const uint32_t blk = blk0 + (uint32_t)i * row_blocks;
          si[i] = a.sidx[blk];
          vv[i] = a.v[blk >> a.group_shift];
        }
      };
      if (s < s1) { fetch_w(s); fetch_x(s); }
      if (!table) {
        for (int i = tid; i < (1 << BITS); i += 64 * QR_WAVES) sh.code[i] = __float_as_uint(a.tables->code[Slot<BITS>::value][i]);
        __syncthreads();
        table = true;
      }
      for (; s < s1; s += QR_WAVES) {
        uint2 cur[8];
        float scale[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if constexpr (BITS == 3) asm("" : "+v"(cw[i].w[0]));         // not at the end of the step before, where it would be waited for
          cur[i] = spread_half<BITS>(cw[i], half);
          if constexpr (BITS == 4) asm("" : "+v"(cur[i].x), "+v"(cur[i].y));   // or the compiler undoes it
          scale[i] = block_scale_by_reciprocal(si[i], vv[i], a.levels, a.inv_levels);
        }
        split_x();
        const int sn = s + QR_WAVES < s1 ? s + QR_WAVES : s;           // past the end: the same step again
        fetch_w(sn); fetch_x(sn);
        for_each_block<QR_SETS>([&](auto set) {
          constexpr int j = decltype(set)::value;
          float w[8];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            w[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sh.code) + code_offset<BITS, j>(cur[i])) * scale[i];
          multiply(w, set);
        });
      }
    } else {
      // four column sets of L1: column 4 c + j of this tile of 64 in set j; columns past Nd count as zero
      const int col = (tile - a.tiles_q) * QR_DCOLS + 4 * c;
      for (; s < s1; s += QR_WAVES) {
        fetch_x(s);
        floatx4 d[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float* p = a.D + (32 * (int64_t)s + 8 * q + i) * a.ldd + col;
          if (a.d_vec) d[i] = col < a.Nd ? *reinterpret_cast<const floatx4*>(p) : floatx4{0.f, 0.f, 0.f, 0.f};
          else {
#pragma unroll
            for (int j = 0; j < 4; ++j) d[i][j] = col + j < a.Nd ? p[j] : 0.f;
          }
        }
        split_x();
        for_each_block<4>([&](auto set) {
          constexpr int j = decltype(set)::value;
          const float w[8] = {d[0][j], d[1][j], d[2][j], d[3][j], d[4][j], d[5][j], d[6][j], d[7][j]};
          multiply(w, set);
        });
      }
    }

    // Sum over the wavefronts in order; wavefront w finishes accumulator register w % 4, i.e. rows 16 t + 4 q + w % 4, of
    // column sets 4 (w / 4) .. + 3.
    const int reg = wave & 3, set0 = 4 * (wave >> 2);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < QR_SETS; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sh.sum[wave][r][j][lane] = acc[t][j][r];
      __syncthreads();
      const int row = row0 + 16 * t + 4 * q + reg;
      floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < QR_WAVES; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] += sh.sum[u][reg][set0 + j][lane];
      if (row >= a.m) continue;
      const int64_t prow = (int64_t)segment * a.m + row;
      if (!dense) {
        const int64_t col = (int64_t)tile * QR_COLS + (NBLK == 2 ? QR_COLS / 8 * set0 + 4 * c : QR_SETS * c + set0);
        if (col < a.N) {
          // X times a scale can leave the range of floats where X times the scaled weights does not (code 0 is 0 whatever the
          // scale): sums that are not finite are formed again from these (24 rows x 4096 x 11008 28.3 -> 28.5 us for looking; a row
          // with NaN 15 us, an infinite one 0.8 ms).
          if constexpr (NBLK > 0)
            if (__builtin_expect(!(fabsf(o[0]) + fabsf(o[1]) + fabsf(o[2]) + fabsf(o[3]) < HUGE_VALF), 0))
              o = plain_sum<BITS>(a, row, col, 32 * (int64_t)s0, 32 * (int64_t)s1);
          *reinterpret_cast<floatx4*>(a.part + prow * a.N + col) = o;
        }
      } else if (set0 == 0) {
        const int col = (tile - a.tiles_q) * QR_DCOLS + 4 * c;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (col + j < a.Nd) a.tpart[prow * a.Nd + col + j] = o[j];
      }
    }
  }
}

// Row tiles of 16 per workgroup (at most QR_TILES, evenly over the workgroups that share a column tile).
static int qrows_tiles(int64_t m) {
  const int64_t tiles = (m + 15) / 16, wgs = (tiles + QR_TILES - 1) / QR_TILES;
  return (int)((tiles + wgs - 1) / wgs);
}

// How the steps are dealt out to the 256 compute units (a constant: it also sizes the workspace, which is asked for without
// a device).  Either every tile is cut into the same number of shares (the steps
// of a tile are counted up to a multiple of the share, so that no share reaches into the next tile), or the shares are
// equal whatever the tiles and some workgroups have two segments, each with its own first fetch and sum: about one and a
// half times a step of all wavefronts.  The smaller number of such steps is taken (4096 x 4096: 7 shares per tile and 3
// steps, 19 us at 24 rows against 24; 4096 x 11008: 6 + 1.5 against 8, 33 us against 36).
struct QrShares { int steps, per_wg, segments; };
static QrShares qrows_shares(int64_t m, int64_t K, int64_t N, int rank) {
  const int rt = qrows_tiles(m);
  const int64_t tiles = (N + QR_COLS - 1) / QR_COLS + (rank + QR_DCOLS - 1) / QR_DCOLS, ksteps = K / 32;
  const int64_t wgs = std::max<int64_t>(1, 256 / ((m + 16 * rt - 1) / (16 * rt)));
  const int64_t even = std::max<int64_t>(1, std::min(wgs / tiles, ksteps / QR_WAVES));
  const int64_t per_even = (ksteps + even - 1) / even;
  const int64_t per_any = std::max<int64_t>((tiles * ksteps + wgs - 1) / wgs, QR_WAVES);
  const double rounds_even = (double)((per_even + QR_WAVES - 1) / QR_WAVES) * (double)((tiles * even + wgs - 1) / wgs);
  const double rounds_any = (double)((per_any + QR_WAVES - 1) / QR_WAVES) + 1.5;
  QrShares s;
  if (rounds_even <= rounds_any) { s.per_wg = (int)per_even; s.steps = (int)(per_even * even); s.segments = (int)even; }
  else { s.per_wg = (int)per_any; s.steps = (int)ksteps; s.segments = (int)((ksteps + per_any - 2) / per_any + 1); }
  return s;
}

size_t qrows_part_floats(int64_t m, int64_t K, int64_t N, int rank) {
  return (size_t)qrows_shares(m, K, N, rank).segments * (size_t)m * (size_t)(N + rank);
}

// Where the form with the scales in X is ahead: figures of whole calls, us, 4096 x 11008 (44 steps per workgroup), rank 64, second form
// -> first, precision 0 / 1.
//              2 bits                    3 bits                    4 bits                    8 bits
//   blocks of 64 (two scales per row of a tile; with three row tiles X times both takes the registers that loads in flight need)
//   12 rows    26.6->20.9 / 20.1->18.1   28.8->23.7 / 21.5->22.1   27.1->21.7 / 20.2->19.3   28.1->23.5 / 22.0->20.9
//   24 rows    29.2->27.9 / 24.6->23.0   30.9->32.0 / 26.0->27.2   29.3->28.8 / 24.1->24.1   30.9->31.2 / 26.5->26.0
//   48 rows    39.8->40.4 / 31.3->32.9   41.0->44.0 / 33.2->35.5   39.2->44.1 / 31.5->32.6   41.1->45.6 / 34.0->37.8
//   blocks of 128 and more
//   12 rows    26.5->19.5 / 20.1->17.2   28.5->21.2 / 21.3->19.6   26.7->20.2 / 20.0->18.4   28.0->22.6 / 21.7->20.2
//   24 rows    29.1->25.6 / 24.5->22.0   30.6->28.1 / 25.9->24.6   28.9->26.9 / 24.0->22.9   30.6->28.8 / 26.3->24.7
//   48 rows    39.3->35.2 / 31.2->29.6   41.1->37.9 / 32.9->33.0   39.2->37.3 / 31.3->31.0   41.0->40.5 / 33.7->32.5
template <int BITS, int RT, bool SPLIT, int NBLK>
constexpr bool scales_in_x_ahead = RT == 1   ? NBLK == 1 || BITS != 3 || SPLIT
                                   : RT == 2 ? NBLK == 1 || BITS == 2 || BITS == 4 || (BITS == 8 && !SPLIT)
                                             : NBLK == 1 && (BITS == 2 || (BITS == 8) != SPLIT);
// A workgroup of that form makes its table first (4 KB for 2 bits, 16 for 3, 64 for 4, 32 for 8): the steps of all wavefronts that
// do not pay it back (24 rows, 4 bits: 19 steps, 4096 x 4096, blocks of 64 16.8 -> 17.6, of 128 16.8 -> 16.6; 27 steps, 5120 x 5120,
// 19.6 -> 20.1 and 19.6 -> 18.6; 2 bits at 19 steps 16.6 -> 16.6 and 16.8 -> 15.7).
template <int BITS, int RT, int NBLK>
constexpr int scaled_rounds = RT == 1 || BITS == 2 ? 2 : NBLK == 2 ? 5 : RT == 2 ? 3 : 4;

template <int BITS, int RT, bool SPLIT, int NBLK>
static bool launch_scaled(const QrArgs& a, dim3 grid, hipStream_t st) {
  if constexpr (scales_in_x_ahead<BITS, RT, SPLIT, NBLK>)
    if (a.per_wg > scaled_rounds<BITS, RT, NBLK> * QR_WAVES) {
      hipLaunchKernelGGL((qrows_kernel<BITS, RT, SPLIT, NBLK>), grid, dim3(64 * QR_WAVES), 0, st, a);
      return true;
    }
  return false;
}
template <int BITS, int RT, bool SPLIT>
static void launch_blocks(const QrArgs& a, dim3 grid, hipStream_t st) {
  if (a.block_shift >= 7 && launch_scaled<BITS, RT, SPLIT, 1>(a, grid, st)) return;
  if (a.block_shift == 6 && launch_scaled<BITS, RT, SPLIT, 2>(a, grid, st)) return;
  hipLaunchKernelGGL((qrows_kernel<BITS, RT, SPLIT, 0>), grid, dim3(64 * QR_WAVES), 0, st, a);
}
template <int BITS, bool SPLIT>
static void launch_rt(const QrArgs& a, int rt, dim3 grid, hipStream_t st) {
  if (rt == 1) launch_blocks<BITS, 1, SPLIT>(a, grid, st);
  else if (rt == 2) launch_blocks<BITS, 2, SPLIT>(a, grid, st);
  else launch_blocks<BITS, 3, SPLIT>(a, grid, st);
}

int launch_qrows(const MvWeights& q, const float* X, int64_t ldx, int64_t K, const float* L1, const float* L2, int64_t ldl2,
                 int rank, int64_t m, int64_t N, int precision, float* Y, int64_t ldy, float* part, size_t part_floats,
                 hipStream_t st) {
  if (m < 1 || m > QROWS_MAX_ROWS || K < 32 || K % 32 || N < 16 || N % 16 || K * N >= (1ll << 31)) return LQ_ERR_SHAPE;
  if (rank < 0 || rank > QROWS_MAX_RANK) return LQ_ERR_RANK;
  if (ldx % 4 || ((uintptr_t)X & 15)) return LQ_ERR_ARG;
  if (q.block < 16 || (q.block & (q.block - 1)) || q.scale_block < 1 || (q.scale_block & (q.scale_block - 1)) || N % q.block)
    return LQ_ERR_CONFIG;
  QrArgs a{};
  a.X = X; a.ldx = ldx; a.codes = q.codes; a.sidx = q.sidx; a.v = q.v;
  a.D = L1; a.ldd = rank; a.Nd = rank;
  a.d_vec = rank % 4 == 0 && ((uintptr_t)L1 & 15) == 0;
  a.K = K; a.N = N; a.m = (int)m;
  const QrShares sh = qrows_shares(m, K, N, rank);
  const int segments = sh.segments;
  a.ksteps = (int)(K / 32); a.steps = sh.steps; a.per_wg = sh.per_wg;
  if (part_floats < (size_t)segments * (size_t)m * (size_t)(N + rank)) return LQ_ERR_WORKSPACE;
  a.tiles_q = (int)((N + QR_COLS - 1) / QR_COLS);
  a.total = a.steps * (a.tiles_q + (rank + QR_DCOLS - 1) / QR_DCOLS);     // K * N is below 2^31
  a.part = part; a.tpart = part + (size_t)segments * (size_t)m * (size_t)N;
  a.block_shift = __builtin_ctz((unsigned)q.block);
  a.group_shift = __builtin_ctz((unsigned)q.scale_block);
  a.levels = q.levels;
  a.inv_levels = 1.0f / (float)q.levels;
  LQ_TRY(device_tables(&a.tables));
  const int rt = qrows_tiles(m);
  const dim3 grid((unsigned)((a.total + a.per_wg - 1) / a.per_wg), (unsigned)((m + 16 * rt - 1) / (16 * rt)));
  {
    prof::Scope ps(prof::QROWS, st, 2.0 * m * (double)K * (double)(N + rank));
#define LQ_QROWS(BITS)                                             \
  case BITS:                                                       \
    if (precision == 0) launch_rt<BITS, true>(a, rt, grid, st);        \
    else launch_rt<BITS, false>(a, rt, grid, st);                      \
    break;
    switch (q.bits) {
      LQ_QROWS(2) LQ_QROWS(3) LQ_QROWS(4) LQ_QROWS(8)
      default: return LQ_ERR_CONFIG;
    }
#undef LQ_QROWS
    LQ_HIP_TRY(hipGetLastError());
  }
  return launch_segment_sum_lowrank(part, a.tpart, m, N, rank, L2, ldl2, Y, ldy, a.steps, a.per_wg, QR_COLS, QR_DCOLS, st);
}

}  // namespace lq
