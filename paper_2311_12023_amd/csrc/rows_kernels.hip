// Forward product with a decomposed weight for 9 to 128 rows of X (decoding many sequences at once, short prompts):
// Y[m x N] = X dequant(codes) + (X L1) L2.  Two launches: the kernel below multiplies X with [Q | L1]
// over ranges of the reduction, qmatvec_finish_kernel or rows_finish_kernel adds the ranges and the product (X L1) L2.
//
// Every weight is decoded (six vector instructions: extract, look up, scale, split into bf16 halves) for at most 48 rows,
// where its matrix instructions take less time than the decode; the codes themselves are 0.25 to 1 byte per weight.  By
// count the decode is a third of the kernel's 20 to 25 us at 24 rows x 4096 x 11008; what bounds it there is the latency of
// loads one step ahead with two wavefronts per SIMD.  Nothing is staged: a lane fetches half a 16-weight run of eight reduction rows, decodes them straight into the
// operand layout of v_mfma_f32_16x16x32_bf16 (8 column sets of 16 columns, column 8 c + j in set j) and multiplies them with
// rows of X that it splits into bf16 halves on the way.  A workgroup owns 128 columns at a time; its eight wavefronts take
// turns at the 32-deep reduction steps and their sums are added in order through LDS.
// Whole call on 4096 x 11008, NF4, rank 64 (4096 x 4096): 24 rows 79 -> 32 us (45 -> 20), 64 rows 84 -> 50 us (47 -> 27),
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
  } else {                                   // bytes 3 half .. 3 half + 2 of six, 2-byte aligned
    const uint16_t* q = reinterpret_cast<const uint16_t*>(run + 2 * half);
    r.w[0] = ((uint32_t)q[0] | ((uint32_t)q[1] << 16)) >> (8 * half);
  }
  return r;
}
// Byte offset of code J's value in the table (4 times the code).  4 bits: the codes are first moved into bytes, four at a
// time, so that a code costs one more instruction instead of a shift and a mask.
template <int BITS>
__device__ __forceinline__ uint2 spread_half(const HalfRun<BITS>& r) {
  if constexpr (BITS == 8) return make_uint2(r.w[0], r.w[1]);
  else if constexpr (BITS == 4) return make_uint2((r.w[0] << 2) & 0x3c3c3c3cu, (r.w[0] >> 2) & 0x3c3c3c3cu);   // even, odd codes
  else return make_uint2(r.w[0] << 2, 0u);
}
template <int BITS, int J>
__device__ __forceinline__ uint32_t code_offset(uint2 r) {
  if constexpr (BITS == 8) return __builtin_amdgcn_ubfe(J < 4 ? r.x : r.y, 8 * (J % 4), 8) << 2;
  else if constexpr (BITS == 4) return __builtin_amdgcn_ubfe(J % 2 ? r.y : r.x, 8 * (J / 2), 8);
  else return (r.x >> (J * BITS)) & (((1u << BITS) - 1u) << 2);
}

// The steps of all column tiles, in order (tile, step), are dealt out in equal contiguous shares, so that every compute unit
// gets the same work whatever the number of tiles; a workgroup's part of a tile is one segment, numbered within the tile.
template <int BITS, int RT, bool SPLIT>
__global__ __launch_bounds__(64 * QR_WAVES, 2) void qrows_kernel(QrArgs a) {
  __shared__ struct {
    float code[1 << BITS];                   // first: a code's offset in the table is its LDS address
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
  auto multiply = [&](const float (&w)[8], auto set) {
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

  bool table = false;
  for (int pos = wg * a.per_wg; pos < end;) {
    const int tile = pos / a.steps, s0 = pos - tile * a.steps;
    int s1 = a.steps - s0 < end - pos ? a.steps : s0 + (end - pos);
    const int segment = wg - (int)((int64_t)tile * a.steps / a.per_wg);
    pos += s1 - s0;
    s1 = s1 < a.ksteps ? s1 : a.ksteps;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int j = 0; j < QR_SETS; ++j) acc[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const bool dense = tile >= a.tiles_q;
    int s = s0 + wave;
    if (!dense) {
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
        for (int i = tid; i < (1 << BITS); i += 64 * QR_WAVES) sh.code[i] = a.tables->code[Slot<BITS>::value][i];
        __syncthreads();
        table = true;
      }
      for (; s < s1; s += QR_WAVES) {
        uint2 cur[8];
        float scale[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          cur[i] = spread_half<BITS>(cw[i]);
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
        const int64_t col = (int64_t)tile * QR_COLS + QR_SETS * c + set0;
        if (col < a.N) *reinterpret_cast<floatx4*>(a.part + prow * a.N + col) = o;
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

template <int BITS, bool SPLIT>
static void launch_rt(const QrArgs& a, int rt, dim3 grid, hipStream_t st) {
  if (rt == 1) hipLaunchKernelGGL((qrows_kernel<BITS, 1, SPLIT>), grid, dim3(64 * QR_WAVES), 0, st, a);
  else if (rt == 2) hipLaunchKernelGGL((qrows_kernel<BITS, 2, SPLIT>), grid, dim3(64 * QR_WAVES), 0, st, a);
  else hipLaunchKernelGGL((qrows_kernel<BITS, 3, SPLIT>), grid, dim3(64 * QR_WAVES), 0, st, a);
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
