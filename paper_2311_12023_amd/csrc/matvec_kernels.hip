// Forward product with a decomposed weight for a handful of input rows (single tokens, small decode batches):
//     Y[m x N] = X[m x K] * dequant(codes)[K x N] + (X * L1)[m x r] * L2[r x N],      m <= 8,
// (Section 3.2 "Implementation", Appendix A: the matrix-vector case of the run-time comparison).  With so few rows the
// product is bound by reading the weights once from HBM (b0/8 bytes each), not by arithmetic, so the weights are decoded
// and multiplied on the vector ALU in fp32: exact products of the same fl32(code * s^) values that Dequantize returns,
// fp32 accumulation.  Two launches: the first multiplies X with [Q | L1] (the columns of L1 are extra column tiles of
// the same grid), the second adds the reduction ranges of both results and the small product (X L1) L2.
//
// Mapping of the first kernel: a thread owns one 16-weight run (one block scale per run, codes fetched as one
// 2..16-byte word) in every 32nd row of its workgroup's range of reduction rows; a workgroup is 8 runs (128 columns) x
// 32 row groups, so that 256 workgroups of up to 512 rows cover a 4096 x 4096 matrix with every load of a thread issued
// before the first is used (the whole matrix is in flight at once, which is what an HBM-bound kernel needs).  The X
// values of the range sit in LDS; they and the code book are asked for before the weights and waited for while those are in
// flight.  Row groups are summed by a fixed butterfly inside each wavefront that deals the columns out on the way, and in
// wavefront order through LDS; the ranges (`splits` of them: enough to fill the machine while the partial sums stay small next to
// the weights) are added in a fixed order by the second kernel, so results are deterministic.
// Whole call on 4096 x 4096, NF4, rank 64: 1 row 13.9 -> 12.0 us, 4 rows 23 -> 16, 8 rows 36 -> 21 (4096 x 11008: 8 rows 58 ->
// 35) by loading before the first barrier, 14 instead of 48 exchanges per row of X, and scales without a division.
// 1 row 13.0 -> 11.2, 8 rows 20.7 -> 18.1 (rank 512: 32.4 -> 21.9 and 49.7 -> 36) by asking for all that the second launch
// reads before it uses any of it.
#include <algorithm>

#include "kernels.h"
#include "nf_device.h"
#include "profiler.h"

namespace lq {

constexpr int MV_RUNS = 8;          // 16-weight runs per workgroup: 128 columns
constexpr int MV_COLS = 16 * MV_RUNS;
constexpr int MV_GROUPS = 32;       // row groups per workgroup (256 threads)
constexpr int MV_ROWS_MAX = 512;    // reduction rows per workgroup (its X slice lives in LDS)
constexpr int MV_DEPTH = MV_ROWS_MAX / MV_GROUPS;   // rows per thread at most

struct MvArgs {
  const float* X; int64_t ldx;      // m x K
  const uint8_t* codes; const uint8_t* sidx; const float* v;   // K x N, row-major flattening
  const float* D; int64_t ldd;      // K x Nd dense (the factor L1), columns tiles_q * 128 onward of the grid
  int d_vec;                        // Nd % 4 == 0 and D 16-byte aligned: float4 loads
  float* Y; int64_t ldy;            // partial sums of X Q: range s at Y + s * m * ldy (splits == 1 and Nd == 0: Y itself)
  float* Yd;                        // partial sums of X D: range s at Yd + s * m * Nd
  int64_t K, N, Nd;
  int m, splits, rows_per_split, tiles_q;
  int block_shift, group_shift, levels;
  float inv_levels;
  const DevTables* tables;
};

template <int BITS, int M>
__global__ __launch_bounds__(256) void qmatvec_kernel(MvArgs a) {
  __shared__ float s_x[M][MV_ROWS_MAX];
  __shared__ float s_code[1 << BITS];
  __shared__ __attribute__((aligned(16))) float s_sum[3][M][MV_COLS];
  const int tid = threadIdx.x, wave = tid >> 6, run = tid & (MV_RUNS - 1), grp = tid >> 3;
  const bool dense = (int)blockIdx.x >= a.tiles_q;                      // a column tile of D instead of the quantized matrix
  const int64_t col = (int64_t)(dense ? blockIdx.x - a.tiles_q : blockIdx.x) * MV_COLS + 16 * run;   // first column of the run
  const int split = blockIdx.y;
  const int64_t ra = (int64_t)split * a.rows_per_split;
  const int64_t rb = ra + a.rows_per_split < a.K ? ra + a.rows_per_split : a.K;
  const int nrows = (int)(rb - ra);
  // the slice of X and the code book are asked for first, then (quantized tiles) all weights of the thread: what waits at
  // the barrier is the former, while the latter are in flight
  float xin[M][MV_ROWS_MAX / 256];
#pragma unroll
  for (int i = 0; i < M; ++i)
#pragma unroll
    for (int h = 0; h < MV_ROWS_MAX / 256; ++h) {
      const int r = tid + 256 * h;
      xin[i][h] = i < a.m && r < nrows ? a.X[(int64_t)i * a.ldx + ra + r] : 0.0f;
    }
  const float book = tid < (1 << BITS) ? a.tables->code[Slot<BITS>::value][tid] : 0.0f;
  auto stage = [&]() {
    if (tid < (1 << BITS)) s_code[tid] = book;
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
      for (int h = 0; h < MV_ROWS_MAX / 256; ++h) s_x[i][tid + 256 * h] = xin[i][h];
    __syncthreads();
  };

  float acc[M][16];
#pragma unroll
  for (int i = 0; i < M; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[i][j] = 0.0f;
  const bool live = col < (dense ? a.Nd : a.N);   // N is a multiple of 16
  const int64_t colc = live ? col : 0;

  if (!dense) {
    // rows of the thread: local rows grp, grp + 32, ...; every load is issued before the first use (a row past the
    // end is loaded clamped and skipped)
    uint2 cw[MV_DEPTH];                           // at most 64 bits of codes per run for b0 <= 4; 8-bit codes take two passes
    uint32_t si[MV_DEPTH];
    float vv[MV_DEPTH];
    constexpr int PASSES = BITS == 8 ? 2 : 1;
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
      for (int j = 0; j < MV_DEPTH; ++j) {
        int r = grp + MV_GROUPS * j;
        r = r < nrows ? r : nrows - 1;
        const int64_t e = (ra + r) * a.N + colc;
        const uint8_t* p = a.codes + (e >> 4) * (2 * BITS) + 8 * pass;
        if constexpr (BITS == 2) cw[j] = make_uint2(*reinterpret_cast<const uint32_t*>(p), 0u);
        else if constexpr (BITS == 3) {
          const uint16_t* q = reinterpret_cast<const uint16_t*>(p);
          cw[j] = make_uint2((uint32_t)q[0] | ((uint32_t)q[1] << 16), (uint32_t)q[2]);
        } else cw[j] = *reinterpret_cast<const uint2*>(p);
        if (pass == 0) {
          const int64_t blk = e >> a.block_shift;
          si[j] = a.sidx[blk];
          vv[j] = a.v[blk >> a.group_shift];
        }
      }
      if (pass == 0) {
        __builtin_amdgcn_sched_barrier(0);
        stage();
      }
      constexpr int PER = 16 / PASSES;            // codes decoded per pass
      constexpr int CB = BITS == 8 ? 8 : BITS;
#pragma unroll
      for (int j = 0; j < MV_DEPTH; ++j) {
        const int r = grp + MV_GROUPS * j;
        if (r < nrows) {
          const float sh = block_scale_by_reciprocal(si[j], vv[j], a.levels, a.inv_levels);
          const uint64_t word = (uint64_t)cw[j].x | ((uint64_t)cw[j].y << 32);
          float xr[M];
#pragma unroll
          for (int i = 0; i < M; ++i) xr[i] = s_x[i][r];
#pragma unroll
          for (int e = 0; e < PER; ++e) {
            const float w = s_code[(uint32_t)(word >> (e * CB)) & ((1u << CB) - 1u)] * sh;
#pragma unroll
            for (int i = 0; i < M; ++i) acc[i][PER * pass + e] = fmaf(xr[i], w, acc[i][PER * pass + e]);
          }
        }
      }
    }
  } else {
    stage();
    // 16 columns of D in the thread's rows, four rows' loads issued together; columns past Nd count as zero
    constexpr int DCH = 4;
    for (int r0 = live ? grp : nrows; r0 < nrows; r0 += DCH * MV_GROUPS) {
      float w[DCH][16];
#pragma unroll
      for (int u = 0; u < DCH; ++u) {
        int r = r0 + u * MV_GROUPS;
        r = r < nrows ? r : nrows - 1;            // loaded clamped, skipped below
        const float* drow = a.D + (ra + r) * a.ldd + col;
        if (a.d_vec) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
            if (col + 4 * q < a.Nd) f = *reinterpret_cast<const float4*>(drow + 4 * q);
            w[u][4 * q] = f.x; w[u][4 * q + 1] = f.y; w[u][4 * q + 2] = f.z; w[u][4 * q + 3] = f.w;
          }
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j) w[u][j] = col + j < a.Nd ? drow[j] : 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < DCH; ++u) {
        const int r = r0 + u * MV_GROUPS;
        if (r < nrows) {
#pragma unroll
          for (int i = 0; i < M; ++i) {
            const float x = s_x[i][r];
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[i][j] = fmaf(x, w[u][j], acc[i][j]);
          }
        }
      }
    }
  }

  // The 8 row groups of a wavefront (lanes 8 apart), by a butterfly that deals the columns out on the way: each step hands
  // half of a lane's columns to its partner, so that row group g of the wavefront ends with columns 2 g' and 2 g' + 1 of its
  // run, g' = g with its bits reversed (14 exchanges per row of X instead of 48).  Then the wavefronts in order through LDS.
  const int lane = tid & 63, gw = lane >> 3;
  const bool b0 = gw & 1, b1 = gw & 2, b2 = gw & 4;
  const int colw = 8 * (int)b0 + 4 * (int)b1 + 2 * (int)b2;      // first of the lane's two columns
  float two[M][2];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    float h8[8], h4[4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float keep = b0 ? acc[i][8 + j] : acc[i][j], give = b0 ? acc[i][j] : acc[i][8 + j];
      h8[j] = keep + dpp_move<0x128>(give);                      // row_ror:8, lanes 8 apart inside a row of 16
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float keep = b1 ? h8[4 + j] : h8[j], give = b1 ? h8[j] : h8[4 + j];
      h4[j] = keep + __shfl_xor(give, 16);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float keep = b2 ? h4[2 + j] : h4[j], give = b2 ? h4[j] : h4[2 + j];
      two[i][j] = keep + __shfl_xor(give, 32);
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < M; ++i)
      *reinterpret_cast<float2*>(&s_sum[wave - 1][i][16 * run + colw]) = make_float2(two[i][0], two[i][1]);
  }
  __syncthreads();
  if (wave == 0 && live) {
    float* __restrict__ Yq = a.Y + (size_t)split * (size_t)a.m * a.ldy;
    float* __restrict__ Yd = a.Yd + (size_t)split * (size_t)a.m * a.Nd;
#pragma unroll
    for (int i = 0; i < M; ++i) {
      if (i >= a.m) break;
      float o[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        float s = two[i][e];
        s += s_sum[0][i][16 * run + colw + e];
        s += s_sum[1][i][16 * run + colw + e];
        s += s_sum[2][i][16 * run + colw + e];
        o[e] = s;
      }
      if (!dense) {
        *reinterpret_cast<float2*>(Yq + (int64_t)i * a.ldy + col + colw) = make_float2(o[0], o[1]);
      } else {
#pragma unroll
        for (int e = 0; e < 2; ++e)
          if (col + colw + e < a.Nd) Yd[(int64_t)i * a.Nd + col + colw + e] = o[e];
      }
    }
  }
}

// Second kernel: Y = sum of the ranges of X Q (in range order) + T L2 with T = sum of the ranges of X L1.  A workgroup
// owns 64 columns and M rows (blockIdx.y picks the rows).  What bounds it is the chain of memory round trips, so everything
// that a rank of 64 needs is asked for before anything is used: the ranges of T and of X Q (thread = (column, slot), rows slot
// and slot + 4; a lane's column is its rank in T), and the rows of L2, of which each of the four slots (one wavefront each) takes a
// quarter for all M rows.  T then goes through LDS to every slot, and the slots' products back to the thread that has the ranges,
// which adds them in slot order.  Both sets of partial sums are described by the distance between ranges and (for T) the
// row pitch, so the kernel also finishes the MFMA path's products of a few dozen rows.
constexpr int MVF_COLS = 64;
constexpr int MVF_SLOTS = 4;
constexpr int MVF_THREADS = MVF_COLS * MVF_SLOTS;
constexpr int MVF_RANK_MAX = 512;
// p[0], p[stride], ...: the first W of n terms, asked for together (past the last: that one again) and added in order.
template <int W>
struct MvfRanges {
  float v[W];
  __device__ __forceinline__ void load(const float* __restrict__ p, size_t stride, int n) {
#pragma unroll
    for (int u = 0; u < W; ++u) v[u] = p[(size_t)(u < n ? u : n - 1) * stride];
  }
  __device__ __forceinline__ float sum(const float* __restrict__ p, size_t stride, int n) const {
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < W; ++u) s += u < n ? v[u] : 0.0f;
    for (int z0 = W; z0 < n; z0 += W) {
      MvfRanges more;
      more.load(p + (size_t)z0 * stride, stride, n - z0);
#pragma unroll
      for (int u = 0; u < W; ++u) s += z0 + u < n ? more.v[u] : 0.0f;
    }
    return s;
  }
};
struct MvfArgs {
  const float* part; size_t pstride; int splits;               // ranges of X Q: range z, row i at part + z * pstride + i * N
  const float* tpart; size_t tstride; int64_t tld; int tsplits;  // ranges of T: row i at tpart + z * tstride + i * tld
  int m; int64_t N; int rank;
  const float* L2; int64_t ldl2;
  float* Y; int64_t ldy;
  // steps != 0: the number of ranges differs between column tiles (see launch_segment_sum_lowrank)
  int steps, per_wg, tile_cols, ttile_cols;
};
// Ranges of a column tile: the workgroups that its steps were dealt to.  Everything the kernel reads waits for this, and the
// steps of all tiles fit 31 bits: divided in 64 bits it took the launch 7.3 instead of 6.0 us
// (24 rows x 4096 x 11008, rank 64; the call 27.1 -> 25.6).
__device__ __forceinline__ int mvf_segments(const MvfArgs& a, uint32_t tile) {
  const uint32_t steps = (uint32_t)a.steps, per_wg = (uint32_t)a.per_wg;
  return (int)(((tile + 1) * steps - 1) / per_wg - tile * steps / per_wg) + 1;
}
// Column tile of the workgroup's columns and the first tile of T.
__device__ __forceinline__ uint32_t mvf_tile(const MvfArgs& a) { return blockIdx.x * (uint32_t)MVF_COLS / (uint32_t)a.tile_cols; }
__device__ __forceinline__ uint32_t mvf_first_ttile(const MvfArgs& a) {
  return a.steps ? ((uint32_t)a.N + (uint32_t)a.tile_cols - 1) / (uint32_t)a.tile_cols : 0u;
}
// RANKS: what LDS holds of T.  Ranks are in flight CHUNK at a time (a lane each).
template <int M, int W, int RANKS>
__global__ __launch_bounds__(MVF_THREADS) void qmatvec_finish_kernel(MvfArgs a) {
  constexpr int CHUNK = RANKS < MVF_COLS ? RANKS : MVF_COLS, PER_SLOT = CHUNK / MVF_SLOTS;
  constexpr int RT = (M + MVF_SLOTS - 1) / MVF_SLOTS;           // rows of a thread
  __shared__ __attribute__((aligned(16))) float s_t[M][RANKS];
  __shared__ float s_sum[MVF_SLOTS][M][MVF_COLS];
  const int tid = threadIdx.x, c = tid % MVF_COLS, slot = __builtin_amdgcn_readfirstlane(tid / MVF_COLS);
  const int64_t col = (int64_t)blockIdx.x * MVF_COLS + c;
  const int row0 = (int)blockIdx.y * M;
  const int m = a.m - row0 < M ? a.m - row0 : M;     // rows of this workgroup
  const bool live = col < a.N;
  const int64_t colc = live ? col : 0;
  const int splits = a.steps ? mvf_segments(a, mvf_tile(a)) : a.splits;
  const uint32_t ttile0 = mvf_first_ttile(a);

  // T, with the tail up to a multiple of a chunk zero: a wavefront has the same rows of it as of X Q, a lane one rank of a chunk
  MvfRanges<W> tv[RT];
  const auto t_from = [&](int i, int p) {
    return a.tpart + (size_t)(row0 + (i < m ? i : m - 1)) * a.tld + (p < a.rank ? p : a.rank - 1);
  };
  const auto t_splits = [&](int p0) { return a.steps ? mvf_segments(a, ttile0 + (uint32_t)p0 / (uint32_t)a.ttile_cols) : a.tsplits; };
  const auto t_load = [&](int p0) {
#pragma unroll
    for (int j = 0; j < RT; ++j)
      if (slot + MVF_SLOTS * j < M) tv[j].load(t_from(slot + MVF_SLOTS * j, p0 + c), a.tstride, t_splits(p0));
  };
  const auto t_store = [&](int p0) {
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const int i = slot + MVF_SLOTS * j;
      if (i >= M) continue;
      const float t = tv[j].sum(t_from(i, p0 + c), a.tstride, t_splits(p0));
      if (c < CHUNK) s_t[i][p0 + c] = p0 + c < a.rank ? t : 0.0f;
    }
  };
  float w[PER_SLOT];
  const auto w_load = [&](int p0) {
#pragma unroll
    for (int u = 0; u < PER_SLOT; ++u) {
      const int q = p0 + PER_SLOT * slot + u;
      w[u] = a.L2[(int64_t)(q < a.rank ? q : a.rank - 1) * a.ldl2 + colc];
    }
  };

  if (a.rank > 0) t_load(0);
  MvfRanges<W> pv[RT];
  const float* prow[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int i = slot + MVF_SLOTS * j;
    prow[j] = a.part + (size_t)(row0 + (i < m ? i : m - 1)) * a.N + colc;
    if (i < M) pv[j].load(prow[j], a.pstride, splits);
  }
  if (a.rank > 0) {
    w_load(0);
    __builtin_amdgcn_sched_barrier(0);
    t_store(0);
    for (int p0 = CHUNK; p0 < a.rank; p0 += CHUNK) { t_load(p0); t_store(p0); }
    __syncthreads();
    float acc[M];
#pragma unroll
    for (int i = 0; i < M; ++i) acc[i] = 0.0f;
    for (int p0 = 0; p0 < a.rank; p0 += CHUNK) {
      float cur[PER_SLOT];
#pragma unroll
      for (int u = 0; u < PER_SLOT; ++u)       // (a row of L2 past the rank counts as zero, whatever was read for it)
        cur[u] = p0 + PER_SLOT * slot + u < a.rank ? w[u] : 0.0f;
      if (p0 + CHUNK < a.rank) w_load(p0 + CHUNK);
#pragma unroll
      for (int i = 0; i < M; ++i)
#pragma unroll
        for (int u = 0; u < PER_SLOT; ++u) acc[i] = fmaf(s_t[i][p0 + PER_SLOT * slot + u], cur[u], acc[i]);
    }
#pragma unroll
    for (int i = 0; i < M; ++i) s_sum[slot][i][c] = acc[i];
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int i = slot + MVF_SLOTS * j;
    if (i >= m) continue;
    float y = pv[j].sum(prow[j], a.pstride, splits);
    if (a.rank > 0) {
#pragma unroll
      for (int u = 0; u < MVF_SLOTS; ++u) y += s_sum[u][i][c];
    }
    if (live) a.Y[(int64_t)(row0 + i) * a.ldy + col] = y;
  }
}

// The same for many rows, where the machine is full and instructions count instead of round trips: a thread takes rows slot and
// slot + 4 through all ranks, 32 loads of a column of L2 at a time, and nothing is exchanged at the end.
// p[0] + p[stride] + ... (n terms, in this order), the loads issued eight at a time.
__device__ __forceinline__ float mvf_range_sum(const float* __restrict__ p, size_t stride, int n) {
  float s = 0.0f;
  for (int z0 = 0; z0 < n; z0 += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = z0 + u < n ? p[(size_t)(z0 + u) * stride] : 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  return s;
}
__global__ __launch_bounds__(MVF_THREADS) void rows_finish_kernel(MvfArgs a) {
  constexpr int M = 8, RT = M / MVF_SLOTS;
  __shared__ float s_t[M][MVF_RANK_MAX];
  const int tid = threadIdx.x, slot = tid / MVF_COLS;
  const int64_t col = (int64_t)blockIdx.x * MVF_COLS + (tid % MVF_COLS);
  const int row0 = (int)blockIdx.y * M;
  const int m = a.m - row0 < M ? a.m - row0 : M;     // rows of this workgroup
  const bool live = col < a.N;
  const int64_t colc = live ? col : 0;
  const int splits = a.steps ? mvf_segments(a, mvf_tile(a)) : a.splits;
  const uint32_t ttile0 = mvf_first_ttile(a);
  // the thread's rows of X Q
  float acc[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int i = slot + MVF_SLOTS * j;
    float s = 0.0f;
    if (i < m) s = mvf_range_sum(a.part + (size_t)(row0 + i) * a.N + colc, a.pstride, splits);
    acc[j] = s;
  }
  // T, with the tail up to a multiple of 32 zero
  const int rank32 = (a.rank + 31) & ~31;
  for (int idx = tid; idx < m * rank32; idx += MVF_THREADS) {
    const int i = idx / rank32, p = idx % rank32;
    float t = 0.0f;
    const int tsplits = a.steps ? mvf_segments(a, ttile0 + (uint32_t)p / (uint32_t)a.ttile_cols) : a.tsplits;
    if (p < a.rank) t = mvf_range_sum(a.tpart + (size_t)(row0 + i) * a.tld + p, a.tstride, tsplits);
    s_t[i][p] = t;
  }
  __syncthreads();
  for (int p0 = 0; p0 < a.rank; p0 += 32) {
    float w[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) w[u] = p0 + u < a.rank ? a.L2[(int64_t)(p0 + u) * a.ldl2 + colc] : 0.0f;
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const int i = slot + MVF_SLOTS * j;
#pragma unroll
      for (int u = 0; u < 32; ++u) acc[j] = fmaf(s_t[i][p0 + u], w[u], acc[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int i = slot + MVF_SLOTS * j;
    if (live && i < m) a.Y[(int64_t)(row0 + i) * a.ldy + col] = acc[j];
  }
}

// Three sizes of T in LDS: with room for 512 ranks where 16 or 64 would do a call takes up to 4 % longer (4096 x 4096, rank 16,
// 8 rows 16.0 -> 16.7 us; rank 64, 1 row 11.1 -> 11.5).
template <int M, int W>
static void launch_finish_w(const MvfArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((a.N + MVF_COLS - 1) / MVF_COLS), (unsigned)((a.m + M - 1) / M));
  if (a.rank <= 16) hipLaunchKernelGGL((qmatvec_finish_kernel<M, W, 16>), grid, dim3(MVF_THREADS), 0, st, a);
  else if (a.rank <= 64) hipLaunchKernelGGL((qmatvec_finish_kernel<M, W, 64>), grid, dim3(MVF_THREADS), 0, st, a);
  else hipLaunchKernelGGL((qmatvec_finish_kernel<M, W, MVF_RANK_MAX>), grid, dim3(MVF_THREADS), 0, st, a);
}
// `ranges`: the most that a value of X Q or of T has.  As many in flight as there are, up to 16: with 8 where there are 16 or more
// a call takes 4 to 26 % longer (4096 x 4096, rank 512, 1 row 21.0 -> 24.4 us; rank 64, 8 rows 16.7 -> 18.0), with 16 where there
// are 3 or 4 up to 19 % (2048 x 28672, rank 64, 8 rows 35.1 -> 36.6, rank 512 50.4 -> 60.2).
template <int M>
static void launch_finish_m(const MvfArgs& a, int ranges, hipStream_t st) {
  if (ranges <= 4) launch_finish_w<M, 4>(a, st);
  else if (ranges <= 8) launch_finish_w<M, 8>(a, st);
  else launch_finish_w<M, 16>(a, st);
}
// Whether rows_finish_kernel is the faster one.  qmatvec_finish_kernel saves round trips, which count while the machine is not
// full, and pays for them with work on ranks past the last (it takes them 64 at a time, the other 32), which counts once it is.
// Measured as whole calls of 9 to 64 rows x 768 to 28672 columns x reductions of 1024 to 8192 x ranks of 8 to 512, 4 bits, by the
// number of workgroups of 8 rows x 64 columns: with the last 64 ranks more than half full and no more of them it is 7 % faster
// up to 256 workgroups, 3 % up to 512, 1.5 % up to 768 and 1 to 4 % slower beyond; with more ranks 8 to 20 %, 3 to 7 %, level, and
// up to 22 % slower; with the last 64 less than half full 1 to 8 % faster up to 256 and slower beyond (ranks above 64), 3 to 6 %
// slower everywhere (17 to 32) or level and slower (up to 16).  Up to 8 rows it is the faster one throughout (4096 x 4096, rank 64,
// 1 row 13.0 -> 11.2 us, 8 rows 20.7 -> 18.2; rank 512 32.4 -> 21.9, 49.7 -> 35.9); what it costs there past 1024 workgroups, at
// one or two rows and ranks just above a multiple of 64, is up to 5 % (1024 x 131072, rank 17, 1 row: 31.7 -> 33.0).
bool rows_finish_preferred(int64_t m, int64_t N, int rank) {
  if (m <= 8) return false;
  if (m > 64 || rank <= 32) return true;
  const int64_t workgroups = (N + MVF_COLS - 1) / MVF_COLS * ((m + 7) / 8);
  return workgroups > ((rank - 1) % 64 < 32 ? 256 : rank <= 64 ? 768 : 512);
}
static int launch_finish(const MvfArgs& a, int ranges, double bytes, hipStream_t st) {
  prof::Scope ps(prof::MISC, st, bytes);
  if (rows_finish_preferred(a.m, a.N, a.rank))
    hipLaunchKernelGGL(rows_finish_kernel, dim3((unsigned)((a.N + MVF_COLS - 1) / MVF_COLS), (unsigned)((a.m + 7) / 8)),
                       dim3(MVF_THREADS), 0, st, a);
  else if (a.m <= 1) launch_finish_m<1>(a, ranges, st);
  else if (a.m <= 2) launch_finish_m<2>(a, ranges, st);
  else if (a.m <= 4) launch_finish_m<4>(a, ranges, st);
  else launch_finish_m<8>(a, ranges, st);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

int launch_range_sum_lowrank(const float* part, size_t pstride, int splits, const float* tpart, size_t tstride,
                             int64_t tld, int tsplits, int64_t m, int64_t N, int rank, const float* L2, int64_t ldl2,
                             float* Y, int64_t ldy, hipStream_t st) {
  if (m < 1 || N < 1 || splits < 1 || rank < 0 || rank > MVF_RANK_MAX || (rank > 0 && tsplits < 1)) return LQ_ERR_SHAPE;
  const MvfArgs a{part, pstride, splits, tpart, tstride, tld, tsplits, (int)m, N, rank, L2, ldl2, Y, ldy, 0, 1, 1, 1};
  return launch_finish(a, std::max(splits, tsplits), 4.0 * ((double)splits * m * (double)N + (double)tsplits * m * rank + (double)rank * (double)N + m * (double)N), st);
}

int launch_segment_sum_lowrank(const float* part, const float* tpart, int64_t m, int64_t N, int rank, const float* L2,
                               int64_t ldl2, float* Y, int64_t ldy, int steps, int per_wg, int tile_cols, int ttile_cols,
                               hipStream_t st) {
  if (m < 1 || N < 1 || rank < 0 || rank > MVF_RANK_MAX || steps < 1 || per_wg < 1 || tile_cols % MVF_COLS || ttile_cols % MVF_COLS ||
      ttile_cols < 1)
    return LQ_ERR_SHAPE;
  const MvfArgs a{part, (size_t)m * (size_t)N, 1, tpart, (size_t)m * (size_t)rank, rank, 1, (int)m, N, rank, L2, ldl2, Y, ldy,
                  steps, per_wg, tile_cols, ttile_cols};
  const double segments = 1.0 + (double)steps / per_wg;
  return launch_finish(a, (steps + per_wg - 2) / per_wg + 1, 4.0 * (segments * m * (double)(N + rank) + (double)rank * (double)N + m * (double)N), st);
}

// Reduction ranges for m rows against K x (N + rank) weights: at most 512 workgroups (with 8 rows two fit a CU, and a
// few more than the machine holds would cost a second round), at most 512 rows each (a multiple of 32), and partial
// sums (splits * m * (N + rank) floats) that stay below about a quarter of a 4-bit matrix's bytes.
int qmatvec_splits(int m, int64_t K, int64_t N, int rank) {
  const int64_t tiles = (N + MV_COLS - 1) / MV_COLS + (rank + MV_COLS - 1) / MV_COLS;
  int64_t s = std::max<int64_t>(1, 512 / tiles);
  s = std::min<int64_t>(s, std::max<int64_t>(1, K / (32 * (int64_t)std::max(m, 1))));
  s = std::max<int64_t>(s, (K + MV_ROWS_MAX - 1) / MV_ROWS_MAX);        // the X slice must fit in LDS
  int64_t rows = (K + s - 1) / s;
  rows = (rows + 31) / 32 * 32;
  return (int)std::max<int64_t>(1, (K + rows - 1) / rows);
}

size_t qmatvec_part_floats(int m, int64_t K, int64_t N, int rank) {
  const int s = qmatvec_splits(m, K, N, rank);
  return (s > 1 || rank > 0) ? (size_t)s * (size_t)m * (size_t)(N + rank) : 0;
}

template <int BITS>
static void launch_m(const MvArgs& a, dim3 grid, hipStream_t st) {
  if (a.m <= 1) hipLaunchKernelGGL((qmatvec_kernel<BITS, 1>), grid, dim3(256), 0, st, a);
  else if (a.m <= 2) hipLaunchKernelGGL((qmatvec_kernel<BITS, 2>), grid, dim3(256), 0, st, a);
  else if (a.m <= 4) hipLaunchKernelGGL((qmatvec_kernel<BITS, 4>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((qmatvec_kernel<BITS, 8>), grid, dim3(256), 0, st, a);
}

int launch_qmatvec(const MvWeights& q, const float* X, int64_t ldx, int64_t K, const float* L1, const float* L2,
                   int64_t ldl2, int rank, int m, int64_t N, float* Y, int64_t ldy, float* part, size_t part_floats,
                   hipStream_t st) {
  if (m < 1 || m > QMATVEC_MAX_ROWS || K <= 0 || N <= 0 || (N % 16) != 0) return LQ_ERR_SHAPE;
  if (rank < 0 || rank > MVF_RANK_MAX) return LQ_ERR_RANK;
  if (q.block < 16 || (q.block & (q.block - 1)) != 0 || q.scale_block < 1 || (q.scale_block & (q.scale_block - 1)) != 0)
    return LQ_ERR_CONFIG;
  if ((N % q.block) != 0 || (ldy & 3) != 0) return LQ_ERR_SHAPE;
  MvArgs a{};
  a.X = X; a.ldx = ldx; a.K = K; a.N = N; a.m = m;
  a.D = L1; a.ldd = rank; a.Nd = rank;
  a.d_vec = (rank > 0 && (rank & 3) == 0 && ((uintptr_t)L1 & 15) == 0) ? 1 : 0;
  a.codes = q.codes; a.sidx = q.sidx; a.v = q.v;
  a.block_shift = __builtin_ctz((unsigned)q.block);
  a.group_shift = __builtin_ctz((unsigned)q.scale_block);
  a.levels = q.levels;
  a.inv_levels = 1.0f / (float)q.levels;
  a.splits = qmatvec_splits(m, K, N, rank);
  int64_t rows = (K + a.splits - 1) / a.splits;
  rows = (rows + 31) / 32 * 32;
  if (rows > MV_ROWS_MAX) return LQ_ERR_SHAPE;
  a.rows_per_split = (int)rows;
  a.splits = (int)((K + rows - 1) / rows);                              // no empty range
  const bool direct = a.splits == 1 && rank == 0;                       // nothing to add afterwards
  if (!direct && part_floats < (size_t)a.splits * (size_t)m * (size_t)(N + rank)) return LQ_ERR_WORKSPACE;
  a.Y = direct ? Y : part;
  a.ldy = direct ? ldy : N;
  a.Yd = direct ? nullptr : part + (size_t)a.splits * (size_t)m * (size_t)N;   // after the partial sums of X Q
  const DevTables* tab = nullptr;
  LQ_TRY(device_tables(&tab));
  a.tables = tab;
  const int64_t tiles_q = (N + MV_COLS - 1) / MV_COLS, tiles_d = (rank + MV_COLS - 1) / MV_COLS;
  if (tiles_q + tiles_d >= (1ll << 31)) return LQ_ERR_SHAPE;
  a.tiles_q = (int)tiles_q;
  const dim3 grid((unsigned)(tiles_q + tiles_d), (unsigned)a.splits);
  {
    // algorithmic bytes: the weights once (codes, one scale index per block, both factors), X, Y
    const double wbytes = (double)K * (double)N * (q.bits / 8.0 + 1.0 / q.block) + 4.0 * (double)rank * (double)(K + N);
    prof::Scope ps(prof::QMATVEC, st, wbytes + 4.0 * m * (double)(K + N));
    switch (q.bits) {
      case 2: launch_m<2>(a, grid, st); break;
      case 3: launch_m<3>(a, grid, st); break;
      case 4: launch_m<4>(a, grid, st); break;
      case 8: launch_m<8>(a, grid, st); break;
      default: return LQ_ERR_CONFIG;
    }
    LQ_HIP_TRY(hipGetLastError());
  }
  if (direct) return LQ_OK;
  return launch_range_sum_lowrank(part, (size_t)m * N, a.splits, a.Yd, (size_t)m * rank, rank, a.splits, m, N, rank, L2,
                                  ldl2, Y, ldy, st);
}

}  // namespace lq
