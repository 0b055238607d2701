// Forward product with a decomposed weight in bf16 for many rows of X (lq_matmul, precision 1):  Y = X Q + (X L1) L2  with
// every operand rounded to bf16 and fp32 accumulation.  The weights are decoded once per call into a bf16 plane that the
// product then reads like any other operand, where qmatmul_kernel decodes a weight again for every 256 rows of X: with one
// MFMA per product that decode cannot hide behind the matrix pipe.  Whole calls, 4 bits, rank 64, without and with a plane: 1500 rows
// x 4096 x 4096 128 -> 92 us, 4096 x 11008 382 -> 229, 11008 x 4096 277 -> 200; 1024 rows 88 -> 75, 199 -> 127, 168 -> 151.
// The line is drawn above 512 rows: 513 rows, with a plane 61, 117, 115 us (4096 x 4096, 4096 x 11008, 11008 x 4096) against 73,
// 196, 137 without; 512 rows 61, 98, 107 against 67, 124, 109, but 8192 x 8192 140 against 133; 256 rows 56, 79, 87 against 56,
// 75, 80 (8192 x 8192 115 against 94).  Small weights: PLANE_M_SMALL in lq_api_matmul.cpp.  The product runs at 1.05 to 1.15 PFLOP/s
// (4096^3 with rank 64: 120 us in a short run, 131 to 133 call after call, at a clock that has come down to 1.8 GHz and 60 % of
// the cycles in the matrix pipe; when it took 156 us: 110 without the MFMAs, 140 without the transfers).
#include <algorithm>

#include "dense_device.h"
#include "kernels.h"
#include "lds_transfer.h"
#include "nf_device.h"
#include "profiler.h"
#include "project_device.h"

namespace lq {

// ------------------------------------------------------------------------------------------------
// Wt[n][k] = bf16(Q[k][n]) and, in the last row of the grid, Lt[n][p] = bf16(L2[p][n]) (p >= rank: zero): a workgroup decodes
// 64 rows x 128 columns, turns them in LDS and writes runs of 64 along k.  Behind these rows of the grid others add the partial
// tiles of T = X L1, which a launch of their own took 5 us for.
constexpr int WP_K = 64, WP_N = 128, WP_PITCH = 33;        // LDS pitch in pairs of bf16

struct WpArgs {
  const uint8_t* codes; const uint8_t* sidx; const float* v;
  const float* L2; int rank, Kd;
  uint16_t* Wt; uint16_t* Lt;
  int64_t K, N, pitch;               // elements from row to row of Wt
  int block_shift, group_shift, levels;
  float inv_levels;
  const DevTables* tables;
  int sum_row;                       // first row of the grid that adds partial tiles of T
  ProjectSum t;
};

template <int BITS>
__global__ __launch_bounds__(256) void weight_plane_kernel(WpArgs a) {
  if ((int)blockIdx.y >= a.sum_row) {
    const int64_t wg = (int64_t)((int)blockIdx.y - a.sum_row) * gridDim.x + blockIdx.x;
    project_sum(a.t, wg * 256 + threadIdx.x, (int64_t)(gridDim.y - a.sum_row) * gridDim.x * 256);
    return;
  }
  __shared__ float s_code[1 << BITS];
  __shared__ uint32_t s_w[WP_N][WP_PITCH];
  const int tid = threadIdx.x, run = tid & 7, pair = tid >> 3;      // two rows 2 pair, 2 pair + 1 of one 16-column run
  const int64_t col = (int64_t)blockIdx.x * WP_N + 16 * run, k0 = (int64_t)blockIdx.y * WP_K;
  const bool low_rank = k0 >= a.K;
  const bool live = col < a.N;                                      // N is a multiple of 16
  float w[2][16];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 16; ++j) w[h][j] = 0.0f;
  if (!low_rank) {
    for (int i = tid; i < (1 << BITS); i += 256) s_code[i] = a.tables->code[Slot<BITS>::value][i];
    uint32_t c[2][16];
    float scale[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int64_t k = k0 + 2 * pair + h;
      k = k < a.K ? k : a.K - 1;                                    // past the end: loaded, never stored
      const int64_t e = k * a.N + (live ? col : 0), blk = e >> a.block_shift;
      load_codes<BITS>(a.codes, e >> 4, c[h]);
      scale[h] = block_scale_by_reciprocal(a.sidx[blk], a.v[blk >> a.group_shift], a.levels, a.inv_levels);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 16; ++j) w[h][j] = s_code[c[h][j]] * scale[h];
  } else if (live) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int p = 2 * pair + h;
      if (p < a.rank) {
#pragma unroll
        for (int j = 0; j < 16; ++j) w[h][j] = a.L2[(int64_t)p * a.N + col + j];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 16; ++j)
    s_w[16 * run + j][pair] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{w[0][j], w[1][j]}, bf16x2));
  __syncthreads();
  uint32_t* out = reinterpret_cast<uint32_t*>(low_rank ? a.Lt : a.Wt);
  const int64_t depth = (low_rank ? a.Kd : a.K) / 2, pitch = (low_rank ? a.Kd : a.pitch) / 2, at = low_rank ? 0 : k0 / 2;   // in pairs
  const int p = tid & 31;
  if (at + p < depth) {
    for (int n = tid >> 5; n < WP_N; n += 8) {
      const int64_t row = (int64_t)blockIdx.x * WP_N + n;
      if (row < a.N) out[row * pitch + at + p] = s_w[n][p];
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Y = A B^T for bf16 planes A (rows x K) and B (columns x K), both with K contiguous, plus a second pair with Kd.  A
// 512-thread workgroup owns a 256 x 256 tile, a wavefront 128 x 64 of it (2 x 4).  Both tiles of a 32-deep step go from
// global memory straight into LDS; four stages, one barrier per step, in the middle of its products: a wavefront waits for its
// own transfers of the next step, the barrier makes that everyone's, and by then all have read the last operands of the
// present stage, which is refilled.  So the operands of each half step are read while the other half multiplies (with the
// barrier between the steps and reads before products the same tiles took 161 instead of 156 us at 4096^3; rows padded
// to spread over the L2's channels changed nothing).  What a wavefront does between its products keeps the matrix pipe waiting,
// since the barrier brings all of them there at once: the loop is unrolled over the stages, so that their addresses are
// constants, the transfers' addresses are carried along instead of worked out (77 -> 30 scalar instructions per step), and the
// transfers go out between the products (4096 x 4096 x 4160 131 -> 120 us, the call 169 -> 162; all four before the operand reads:
// 2 to 4 % more, but less where the weights come from memory and rows begin inside a line, which they no longer do).  Rows are 64 bytes, unit u of a
// row stored at u ^ ((row / 4) % 4): 16 lanes' reads of 128 bits fall into different banks (with (row / 2) % 4 into half of
// them, twice the LDS cycles; 0.6 % of the call, in qmatmul_kernel 0.3 %).
constexpr int PG_T = 256, PG_STAGES = 4, PG_THREADS = 512;
constexpr uint32_t PG_TILE = PG_T * 64, PG_STAGE = 2 * PG_TILE;            // bytes

struct PgArgs {
  const uint16_t* A; const uint16_t* B; int64_t pitch;      // elements from row to row
  const uint16_t* A2; const uint16_t* B2; int64_t pitch2;
  float* Y; int64_t ldy;             // splits == 1: m x N; else range s at Y + s * m * ldy
  int64_t m, N;
  int nsteps1, nsteps, splits, tiles_m, tiles_n;
};

__global__ __launch_bounds__(PG_THREADS) void plane_gemm_kernel(PgArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char pg_lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int ln = lane & 31, lh = lane >> 5;
  // (tile, range) pairs are dealt to the 8 XCDs in contiguous stretches, tiles in an order that goes down four row tiles before
  // the next column, so that the tiles an XCD works on at a time share operands in its L2.  Pairs and not tiles, or a few
  // tiles of many ranges fill some XCDs twice and leave others idle (1025 rows x 4096 x 1024, 20 tiles of 12 ranges)
  const int items = a.tiles_m * a.tiles_n * a.splits, per = (items + 7) / 8;
  const int item = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || item >= items) return;
  const int t = item / a.splits, split = item - t * a.splits;
  const int band = t / (4 * a.tiles_n), rows = a.tiles_m - 4 * band < 4 ? a.tiles_m - 4 * band : 4;
  const int inside = t - band * 4 * a.tiles_n;
  const int tm = 4 * band + inside % rows, tn = inside / rows;
  const int s0 = (int)((int64_t)a.nsteps * split / a.splits), s1 = (int)((int64_t)a.nsteps * (split + 1) / a.splits);

  // this wavefront's transfers: rows 16 wave .. + 15 and 128 further of both tiles; lane l brings unit l % 4 ^ swizzle of row l / 4
  const int lrow = lane >> 2, unit = (lane & 3) ^ ((lrow >> 2) & 3);
  const uint32_t voff1 = (uint32_t)(lrow * a.pitch * 2 + unit * 16), voff2 = (uint32_t)(lrow * a.pitch2 * 2 + unit * 16);
  const int64_t arow = (int64_t)tm * PG_T + 16 * wave, brow = (int64_t)tn * PG_T + 16 * wave;
  // Where the next step's transfers read: this wavefront's rows of the present pair of planes at the present reduction index.
  const uint16_t *pa, *pb;
  int64_t rows128;                               // elements to the rows 128 further
  uint32_t voff;
  int next = s0;                                 // the step that these belong to
  auto plane_pair = [&](bool second, int64_t k) {
    const int64_t pitch = second ? a.pitch2 : a.pitch;
    pa = (second ? a.A2 : a.A) + arow * pitch + k;
    pb = (second ? a.B2 : a.B) + brow * pitch + k;
    rows128 = 128 * pitch;
    voff = second ? voff2 : voff1;
  };
  plane_pair(s0 >= a.nsteps1, 32 * (int64_t)(s0 >= a.nsteps1 ? s0 - a.nsteps1 : s0));
  auto transfer = [&](int part, int stage) {     // a quarter of a step's transfers
    const uint32_t lds = (uint32_t)stage * PG_STAGE + (uint32_t)wave * 1024u + 8192u * part;
    transfer_to_lds((part < 2 ? pa : pb) + (part & 1 ? rows128 : 0), voff, lds);
  };
  auto advance = [&]() {                         // past the end: the last step again, into a stage that nobody reads any more
    if (next + 1 >= s1) return;
    ++next;
    if (next == a.nsteps1) plane_pair(true, 0);
    else { pa += 32; pb += 32; }
  };

  floatx16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  const int wm = wave >> 2, wn = wave & 3;
  // operand addresses for the two 16-deep halves of a step; a row tile is 2 KB further
  uint32_t aoff[2], boff[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const uint32_t u = (uint32_t)((2 * g + lh) ^ ((ln >> 2) & 3)) * 16u;
    aoff[g] = (uint32_t)(128 * wm + ln) * 64u + u;
    boff[g] = PG_TILE + (uint32_t)(64 * wn + ln) * 64u + u;
  }

  bf16x8 x[2][4], b[2][2];                       // operands of the two halves of a step
  auto read = [&](int stage, int g) __attribute__((always_inline)) {
    const unsigned char* from = pg_lds + (uint32_t)stage * PG_STAGE;
#pragma unroll
    for (int j = 0; j < 2; ++j) b[g][j] = *reinterpret_cast<const bf16x8*>(from + boff[g] + 2048u * j);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[g][i] = *reinterpret_cast<const bf16x8*>(from + aoff[g] + 2048u * i);
    __builtin_amdgcn_sched_barrier(0);           // the reads go out before the products of the other half
  };
  auto multiply = [&](int g, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[g][i], b[g][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int p = 0; p < PG_STAGES; ++p) {
#pragma unroll
    for (int part = 0; part < 4; ++part) transfer(part, p);
    advance();
  }
  asm volatile("s_waitcnt vmcnt(12)\n\ts_barrier" ::: "memory");   // 4 transfers a step: the first step's are done
  read(0, 0);
  auto step = [&](auto stage) __attribute__((always_inline)) {
    constexpr int u = decltype(stage)::value;
    read(u, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) multiply(0, i);
    // the next step has arrived when at most the transfers of the two steps after it are outstanding; past the barrier that
    // holds for every wavefront, and none reads this stage any more
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    read((u + 1) % PG_STAGES, 0);                // past the end: never used (a branch here would cost exact waits)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      multiply(1, i);
      transfer(i, u);
      __builtin_amdgcn_sched_barrier(0);
    }
    advance();
  };
  int s = s0;
  for (; s + PG_STAGES <= s1; s += PG_STAGES) for_each_block<PG_STAGES>(step);
  for_each_block<PG_STAGES - 1>([&](auto stage) { if (s + decltype(stage)::value < s1) step(stage); });
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // nothing lands in LDS after the workgroup is gone

  float* __restrict__ Y = a.Y + (size_t)split * (size_t)a.m * (size_t)a.ldy;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int64_t col = (int64_t)tn * PG_T + 64 * wn + 32 * j + ln;
    if (col >= a.N) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int64_t row = (int64_t)tm * PG_T + 128 * wm + 32 * i + 8 * (e >> 2) + 4 * lh + (e & 3);
        if (row < a.m) Y[row * a.ldy + col] = acc[i][j][e];
      }
  }
}

size_t weight_plane_elems(int64_t pitch, int64_t N) { return (size_t)((N + PG_T - 1) / PG_T * PG_T) * (size_t)pitch; }

template <int BITS>
static void launch_weight_plane(const WpArgs& a, dim3 grid, hipStream_t st) {
  hipLaunchKernelGGL(weight_plane_kernel<BITS>, grid, dim3(256), 0, st, a);
}

int launch_plane_product(const MvWeights& q, const uint16_t* Xh, int64_t K, const uint16_t* Th, int Kd, const float* L2,
                         int rank, int64_t m, int64_t rows_pad, int64_t N, uint16_t* Wt, uint16_t* Lt, float* Y, int64_t ldy,
                         float* part, size_t part_floats, const ProjectSum& t, hipStream_t st) {
  if (m < 1 || rows_pad < m || rows_pad % PG_T || K < 32 || K % 32 || N < 16 || N % 16 || K * N >= (1ll << 31) ||
      rows_pad * K >= (1ll << 31))
    return LQ_ERR_SHAPE;
  if (rank < 0 || (rank > 0 && (Kd < rank || Kd % 32 || Kd > WP_K))) return LQ_ERR_RANK;
  if (q.block < 16 || (q.block & (q.block - 1)) || q.scale_block < 1 || (q.scale_block & (q.scale_block - 1)) || N % q.block)
    return LQ_ERR_CONFIG;
  WpArgs w{};
  w.codes = q.codes; w.sidx = q.sidx; w.v = q.v; w.L2 = L2; w.rank = rank; w.Kd = Kd; w.Wt = Wt; w.Lt = Lt; w.K = K; w.N = N; w.pitch = plane_pitch(K);
  w.block_shift = __builtin_ctz((unsigned)q.block);
  w.group_shift = __builtin_ctz((unsigned)q.scale_block);
  w.levels = q.levels;
  w.inv_levels = 1.0f / (float)q.levels;
  LQ_TRY(device_tables(&w.tables));
  const int64_t wx = (N + WP_N - 1) / WP_N, wy = (K + WP_K - 1) / WP_K + (rank > 0 ? 1 : 0);
  const int64_t sum_wgs = t.splits > 0 ? (t.rows_pad * (t.Kd >> 2) + 255) / 256 : 0;
  const int64_t sum_rows = std::min<int64_t>((std::min<int64_t>(sum_wgs, 4096) + wx - 1) / wx, 65535 - wy);
  if (wy > 65535 || (sum_wgs > 0 && sum_rows < 1)) return LQ_ERR_SHAPE;
  w.sum_row = (int)wy; w.t = t;
  const dim3 wgrid((unsigned)wx, (unsigned)(wy + sum_rows));
  {
    prof::Scope ps(prof::WEIGHT_PLANE, st, (double)K * (double)N * (q.bits / 8.0 + 2.0));
    switch (q.bits) {
      case 2: launch_weight_plane<2>(w, wgrid, st); break;
      case 3: launch_weight_plane<3>(w, wgrid, st); break;
      case 4: launch_weight_plane<4>(w, wgrid, st); break;
      case 8: launch_weight_plane<8>(w, wgrid, st); break;
      default: return LQ_ERR_CONFIG;
    }
    LQ_HIP_TRY(hipGetLastError());
  }
  PgArgs a{};
  a.A = Xh; a.B = Wt; a.pitch = plane_pitch(K); a.A2 = Th; a.B2 = Lt; a.pitch2 = rank > 0 ? Kd : 0;
  a.m = m; a.N = N;
  a.nsteps1 = (int)(K / 32);
  a.nsteps = a.nsteps1 + (int)(a.pitch2 / 32);
  a.tiles_m = (int)((m + PG_T - 1) / PG_T);
  a.tiles_n = (int)((N + PG_T - 1) / PG_T);
  a.splits = qmatmul_splits(m, N, a.nsteps);
  if (a.splits > 1 && part_floats < (size_t)a.splits * (size_t)m * (size_t)N) return LQ_ERR_WORKSPACE;
  a.Y = a.splits > 1 ? part : Y;
  a.ldy = a.splits > 1 ? N : ldy;
  const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
  if (tiles >= (1ll << 28)) return LQ_ERR_SHAPE;
  constexpr size_t lds = (size_t)PG_STAGES * PG_STAGE;
  static LdsLimit limit;
  LQ_TRY(limit.raise(reinterpret_cast<const void*>(plane_gemm_kernel), lds));
  {
    prof::Scope ps(prof::PLANE_GEMM, st, 2.0 * (double)m * (double)N * (double)(K + a.pitch2));
    hipLaunchKernelGGL(plane_gemm_kernel, dim3((unsigned)((tiles * a.splits + 7) / 8 * 8)), dim3(PG_THREADS), lds, st, a);
    LQ_HIP_TRY(hipGetLastError());
  }
  if (a.splits > 1) return launch_qmatmul_reduce(part, a.splits, m, N, Y, ldy, st);
  return LQ_OK;
}

}  // namespace lq
