// The large products of the randomized SVD's cold start, one problem at a time (see gemm_kernels.hip for the operands and
// for batches): C[l x M] = X A^T and C[l x N] = X A with fp32 A and the reduction dealt out to the wavefronts of a workgroup.
#include <algorithm>
#include <cmath>

#include "dense_device.h"
#include "kernels.h"
#include "mfma_device.h"
#include "profiler.h"

namespace lq {

// A workgroup owns l rows x 16 NT columns of the result and a range of the reduction, whose 32-deep steps its four wavefronts
// take in turn.  Every operand goes from memory into the registers of the one wavefront that multiplies it, on
// v_mfma_f32_16x16x32_bf16 (both sides split into bf16 hi + lo, three products each, fp32 accumulation): the loop has
// neither barriers nor LDS traffic, and a row of a step of A is one 128-byte line.  X comes packed in operand layout, so that a step of it is one contiguous stretch (as rows 16 KB apart it took the
// kernel three times as long: the lines of a step then share an L2 channel).  The four partial results are added in LDS in
// wavefront order.  Where the column tiles do not fill the chip the reduction is also cut into ranges, whose sums lie in
// `part` (columns past the result are zero there) and are added, in order, by whoever reads the product next
// (column_sum_kernel, filter_step_kernel): partial sums amount to a few results, where 256-column tiles needed 16.
// What bounds it: L2, X being read once per tile (at 4096 columns and l = 128 half a megabyte beside a quarter of A per
// compute unit), and below that the length of a single pass through memory.  With one wavefront per SIMD a load that waits for its
// turn holds up the products behind it, so loads, split and products alternate row block by row block (24 loads, the split
// and then 96 products per step took l = 128, 4096 x 4096 23.3 (X A) and 22.1 us, 4096 x 11008 56.4 and 48.1; now 18.5 and 21.4,
// 44.3 and 44.6).  Beginning at another step in every tile, against rows of A that share an L2 channel, changed nothing.  Measured with the launches
// that split X and add the ranges, against the kernel for batches and its fix-up (us, X A^T / X A): l = 64, 768 x 768 20.0 /
// 17.5 -> 8.7 / 8.5; l = 96, 2500 x 4096 27.9 / 26.3 -> 23 / 22; l = 128, 4096 x 4096 40.2 / 38.5 -> 34.7 / 31.9, 4096 x 11008
// 76.5 / 67.3 -> 71.5 / 59.8; where the neighbouring kernels split and add, 4 to 8 us less.  As the cold start runs them: l = 128,
// 8192 x 8192 97 / 86 -> 69 / 69, 8192 x 28672 308 / 259 -> 257 / 255, 28672 x 8192 312 / 264 -> 279 / 227; l = 32, 512 x 512 17.3 / 14.4 ->
// 4.3 / 4.2, 4096 x 4096 23.6 / 22.3 -> 18.6 / 22.4, 8192 x 28672 229 / 181 -> 173 / 193 (the one loss, less than its other product
// gains: factorizations there take 0.93 of the time).  Twenty shapes of factorizations take 0.53 to 0.93 of the time.
constexpr int COL_THREADS = 256, COL_BK = 32;

struct ColArgs {
  const uintx4* X;
  const float* A;
  int64_t lda, big, K;
  int ns, per_range, ranges;     // steps of the reduction, of a range, number of ranges
  float* part; int64_t ldp;      // ranges > 1: range r of row i at part + (r l + i) ldp
  float* C; int64_t ldc;         // ranges == 1: the result (NULL: not wanted), and in operand layout (NULL: not wanted)
  uintx2* packed;
};

template <int N> struct Words;
template <> struct Words<1> { typedef float type; };
template <> struct Words<2> { typedef floatx2 type; };
template <> struct Words<4> { typedef floatx4 type; };

// What a step needs of A: column j, k = 16 h + 4 q + 0..3 (NT mode); row e, k = e < 4 ? 4 q + e : 12 + 4 q + e, of NT columns (NN).
template <int MODE, int NT> struct ColA;
template <int NT> struct ColA<MODE_NT, NT> { floatx4 v[NT][2]; };
template <int NT> struct ColA<MODE_NN, NT> { typename Words<NT>::type v[8]; };
template <int LB> struct ColX { uintx4 v[LB][2]; };

// off: byte offset of the lane's elements of column j (NT mode), of its columns in its first row (NN mode: off[0]).  TAIL:
// elements past the end of the reduction count as zero and are not read.
template <int MODE, int NT, bool TAIL>
__device__ __forceinline__ void col_fetch_a(const float* A, int64_t lda, int64_t K, const uint32_t (&off)[MODE == MODE_NT ? NT : 1],
                                            int q, int64_t k0, ColA<MODE, NT>& a) {
  if constexpr (MODE == MODE_NT) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        floatx4 w = {0.f, 0.f, 0.f, 0.f};
        if (!TAIL || k0 + 16 * h + 4 * q < K) w = *reinterpret_cast<const floatx4*>(reinterpret_cast<const char*>(A + k0 + 16 * h) + off[j]);
        a.v[j][h] = w;
      }
  } else {
    typedef typename Words<NT>::type Row;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = e < 4 ? e : 12 + e;
      Row w = Row(0.f);
      if (!TAIL || k0 + k + 4 * q < K) w = *reinterpret_cast<const Row*>(reinterpret_cast<const char*>(A + (size_t)(k0 + k) * lda) + off[0]);
      a.v[e] = w;
    }
  }
}

template <int LB>
__device__ __forceinline__ void col_fetch_x(const uintx4* X, int lane, int64_t k0, ColX<LB>& x) {
  const uintx4* base = X + (size_t)(k0 / COL_BK) * (LB * 2 * 64);
#pragma unroll
  for (int i = 0; i < LB; ++i)
#pragma unroll
    for (int p = 0; p < 2; ++p) x.v[i][p] = base[(2 * i + p) * 64 + lane];
}

// Load n of a step's A (NT mode: 2 NT of them, NN: 8); a step inside the reduction.
template <int MODE, int NT> constexpr int COL_A_LOADS = MODE == MODE_NT ? 2 * NT : 8;
template <int MODE, int NT>
__device__ __forceinline__ void col_fetch_a_part(const float* A, int64_t lda, const uint32_t (&off)[MODE == MODE_NT ? NT : 1], int64_t k0, int n,
                                                 ColA<MODE, NT>& a) {
  if constexpr (MODE == MODE_NT) {
    a.v[n >> 1][n & 1] = *reinterpret_cast<const floatx4*>(reinterpret_cast<const char*>(A + k0 + 16 * (n & 1)) + off[n >> 1]);
  } else {
    typedef typename Words<NT>::type Row;
    a.v[n] = *reinterpret_cast<const Row*>(reinterpret_cast<const char*>(A + (size_t)(k0 + (n < 4 ? n : 12 + n)) * lda) + off[0]);
  }
}

// A's operands of a step: bf16 high and low halves.  Pair n (of 4 NT): elements 2 (n % 4), 2 (n % 4) + 1 of column n / 4.
template <int NT> struct ColOps { bf16x8 h[NT], l[NT]; };
template <int MODE, int NT>
__device__ __forceinline__ void col_split_pair(const ColA<MODE, NT>& a, int n, ColOps<NT>& o) {
  const int j = n >> 2, e = 2 * (n & 3);
  floatx2 v;
  if constexpr (MODE == MODE_NT) v = floatx2{a.v[j][e >> 2][e & 3], a.v[j][e >> 2][(e & 3) + 1]};
  else if constexpr (NT == 1) v = floatx2{a.v[e], a.v[e + 1]};
  else v = floatx2{a.v[e][j], a.v[e + 1][j]};
  bf16x2 h, l;
  split_bf16(v, h, l);
  o.h[j][e] = h[0]; o.h[j][e + 1] = h[1]; o.l[j][e] = l[0]; o.l[j][e + 1] = l[1];
}
template <int MODE, int NT>
__device__ __forceinline__ void col_split(const ColA<MODE, NT>& a, ColOps<NT>& o) {
#pragma unroll
  for (int n = 0; n < 4 * NT; ++n) col_split_pair<MODE, NT>(a, n, o);
}
template <int NT>
__device__ __forceinline__ void col_multiply_row(const uintx4 (&x)[2], const ColOps<NT>& o, floatx4 (&acc)[NT]) {
  const bf16x8 xh = __builtin_bit_cast(bf16x8, x[0]), xl = __builtin_bit_cast(bf16x8, x[1]);
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, o.h[j], acc[j], 0, 0, 0);
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, o.l[j], acc[j], 0, 0, 0);
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, o.h[j], acc[j], 0, 0, 0);
}

// LB = l / 16.  Large accumulators: one wavefront per SIMD with all its registers.
template <int LB, int MODE, int NT>
__global__ __launch_bounds__(COL_THREADS, LB * NT <= 8 ? 2 : 1) void column_gemm_kernel(ColArgs g) {
  extern __shared__ __attribute__((aligned(16))) float sums[];            // [wavefront][LB][NT][64 lanes][4]
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int range = blockIdx.x % g.ranges, tile = blockIdx.x / g.ranges;  // the ranges of X are dealt to the XCDs
  const int64_t big0 = (int64_t)tile * (16 * NT);
  uint32_t off[MODE == MODE_NT ? NT : 1];
  if constexpr (MODE == MODE_NT) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int64_t row = std::min<int64_t>(big0 + NT * n + j, g.big - 1);          // what is clamped is never part of the result
      off[j] = (uint32_t)((row * g.lda + 4 * q) * 4);
    }
  } else {
    const int64_t col = std::min<int64_t>(big0 + NT * n, g.big - NT);               // big is a multiple of NT
    off[0] = (uint32_t)(((int64_t)4 * q * g.lda + col) * 4);
  }
  // This wavefront's steps are s0 + w, s0 + w + 4, ..; a partial last step of the reduction follows after the loop, which
  // therefore holds no guarded load; prefetches past the end read the last step again.
  const int s0 = range * g.per_range, s1 = std::min(s0 + g.per_range, g.ns), full = (int)(g.K / COL_BK);
  const int last = std::min(s1, full), count = last > s0 + w ? (last - s0 - w + 3) / 4 : 0;
  const int64_t kfirst = (int64_t)(s0 + w) * COL_BK;

  floatx4 acc[LB][NT];
#pragma unroll
  for (int i = 0; i < LB; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  ColA<MODE, NT> a[2];
  ColX<LB> x[2];
  ColOps<NT> o[2];
  if (count > 0) {
    auto at = [&](int t) { return kfirst + (int64_t)(t < count ? t : count - 1) * (4 * COL_BK); };
    auto first = [&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      col_fetch_a<MODE, NT, false>(g.A, g.lda, g.K, off, q, at(0), a[u]);
      col_fetch_x<LB>(g.X, lane, at(0), x[u]);
      col_fetch_a<MODE, NT, false>(g.A, g.lda, g.K, off, q, at(1), a[1 - u]);
      __builtin_amdgcn_sched_barrier(0);
      col_split<MODE, NT>(a[u], o[u]);
    };
    // Row block by row block: the products, between them the loads of X for the next step and of A for the one after it and the
    // split of A for the next, so that the loads do not queue up in front of the products.
    auto step = [&](auto uc, int t) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value, NA = COL_A_LOADS<MODE, NT>;
      const int64_t k1 = at(t + 1), k2 = at(t + 2);
      const uintx4* xnext = g.X + (size_t)(k1 / COL_BK) * (LB * 2 * 64) + lane;
#pragma unroll
      for (int i = 0; i < LB; ++i) {
#pragma unroll
        for (int p = 0; p < 2; ++p) x[(u + 1) % 2].v[i][p] = xnext[(2 * i + p) * 64];
#pragma unroll
        for (int n = i * NA / LB; n < (i + 1) * NA / LB; ++n) col_fetch_a_part<MODE, NT>(g.A, g.lda, off, k2, n, a[u % 2]);
#pragma unroll
        for (int n = i * 4 * NT / LB; n < (i + 1) * 4 * NT / LB; ++n) col_split_pair<MODE, NT>(a[(u + 1) % 2], n, o[(u + 1) % 2]);
        col_multiply_row<NT>(x[u % 2].v[i], o[u % 2], acc[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // An odd step goes first: behind the loop the accumulators would be copied in every round of it.
    const std::integral_constant<int, 0> even{};
    const std::integral_constant<int, 1> odd{};
    int t = count & 1;
    if (t) { first(odd); step(odd, 0); }
    else first(even);
    for (; t < count; t += 2) { step(even, t); step(odd, t + 1); }
  }
  if (s1 == g.ns && full < g.ns && s0 <= full && (full - s0) % 4 == w) {
    col_fetch_a<MODE, NT, true>(g.A, g.lda, g.K, off, q, (int64_t)full * COL_BK, a[0]);
    col_fetch_x<LB>(g.X, lane, (int64_t)full * COL_BK, x[0]);
    col_split<MODE, NT>(a[0], o[0]);
#pragma unroll
    for (int i = 0; i < LB; ++i) col_multiply_row<NT>(x[0].v[i], o[0], acc[i]);
  }

  floatx4* mine = reinterpret_cast<floatx4*>(sums) + (size_t)w * (LB * NT * 64) + lane;
#pragma unroll
  for (int i = 0; i < LB; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) mine[(i * NT + j) * 64] = acc[i][j];
  __syncthreads();
  // A thread takes four consecutive columns of a row; element r of a lane's accumulator is row 4 q + r, column NT n + j.
  for (int idx = threadIdx.x; idx < 16 * LB * 4 * NT; idx += COL_THREADS) {
    const int row = idx / (4 * NT), c4 = 4 * (idx % (4 * NT));
    const int64_t col = big0 + c4;
    floatx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n1 = (c4 + e) / NT, j1 = (c4 + e) % NT;
      const float* p = sums + ((((row >> 4) * NT + j1) * 64 + 16 * ((row & 15) >> 2) + n1) * 4 + (row & 3));
      v[e] = col + e < g.big ? ((p[0] + p[LB * NT * 256]) + p[2 * LB * NT * 256]) + p[3 * LB * NT * 256] : 0.f;
    }
    if (g.ranges > 1) {
      *reinterpret_cast<floatx4*>(g.part + ((size_t)range * (16 * LB) + row) * g.ldp + col) = v;
    } else {
      if (g.packed) store_packed(g.packed, LB, row, col, v);
      if (g.C) {
        float* o = g.C + (size_t)row * g.ldc + col;
        if (col + 4 <= g.big) *reinterpret_cast<floatx4*>(o) = v;
        else for (int e = 0; col + e < g.big; ++e) o[e] = v[e];
      }
    }
  }
}

// Sum of the ranges of a product, in order (ranges == 1: a matrix as it is), as fp32 to C and in operand layout to packed
// (either may be NULL).  Sixteen rows and 64 columns per workgroup, so that it writes whole lines of either.
__global__ __launch_bounds__(256) void column_sum_kernel(const float* __restrict__ src, int64_t ld, int ranges, float* __restrict__ C,
                                                         int64_t ldc, int64_t big, uintx2* __restrict__ packed) {
  const int64_t col = (int64_t)blockIdx.x * 64 + 4 * (threadIdx.x & 15);
  const int row = blockIdx.y * 16 + (threadIdx.x >> 4);
  const float* p = src + (size_t)row * ld + col;
  const size_t next = (size_t)(16 * gridDim.y) * ld;
  floatx4 v = *reinterpret_cast<const floatx4*>(p);
#pragma unroll 4
  for (int r = 1; r < ranges; ++r) v += *reinterpret_cast<const floatx4*>(p + r * next);
  if (packed) store_packed(packed, gridDim.y, row, col, v);
  if (C) {
    float* o = C + (size_t)row * ldc + col;
    if (col + 4 <= big) *reinterpret_cast<floatx4*>(o) = v;
    else for (int e = 0; col + e < big; ++e) o[e] = v[e];
  }
}

int launch_column_sum(int l, const float* src, int64_t ld, int ranges, int64_t big, float* C, int64_t ldc, uint16_t* packed,
                      hipStream_t st) {
  if (l % 16 || l < 16 || ld < 64 || ld % 64 || ranges < 1) return LQ_ERR_ARG;
  if (ld / 64 >= (1ll << 31)) return LQ_ERR_SHAPE;
  prof::Scope ps(prof::COLUMN_SUM, st, 4.0 * l * ld * (ranges + (C ? 1 : 0) + (packed ? 1 : 0)));
  hipLaunchKernelGGL(column_sum_kernel, dim3((unsigned)(ld / 64), (unsigned)(l / 16)), dim3(256), 0, st, src, ld, ranges, C, ldc, big,
                     reinterpret_cast<uintx2*>(packed));
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

template <int LB, int MODE, int NT>
static int launch_tile(const ColArgs& g, int64_t tiles, hipStream_t st) {
  constexpr size_t lds = (size_t)4 * LB * NT * 64 * sizeof(floatx4);
  if constexpr (lds > 65536) {
    static LdsLimit limit;
    LQ_TRY(limit.raise(reinterpret_cast<const void*>(column_gemm_kernel<LB, MODE, NT>), lds));
  }
  hipLaunchKernelGGL((column_gemm_kernel<LB, MODE, NT>), dim3((unsigned)(tiles * g.ranges)), dim3(COL_THREADS), lds, st, g);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

template <int LB, int MODE>
static int launch_width(const ColArgs& g, int nt, int64_t tiles, hipStream_t st) {
  return nt == 1 ? launch_tile<LB, MODE, 1>(g, tiles, st) : nt == 2 ? launch_tile<LB, MODE, 2>(g, tiles, st) : launch_tile<LB, MODE, 4>(g, tiles, st);
}

template <int MODE>
static int launch_rows(const ColArgs& g, int l, int nt, int64_t tiles, hipStream_t st) {
  switch (l / 16) {
    case 2: return launch_width<2, MODE>(g, nt, tiles, st);
    case 4: return launch_width<4, MODE>(g, nt, tiles, st);
    case 6: return launch_width<6, MODE>(g, nt, tiles, st);
    case 8: return launch_width<8, MODE>(g, nt, tiles, st);
    default: return LQ_ERR_ARG;
  }
}

bool column_gemm_supported(int l) { return l % 32 == 0 && l >= 32 && l <= 128; }

// Width of the tiles (16 nt columns) and number of ranges by what a launch is estimated to take, in us: per round of 256
// workgroups what each reads (X out of L2 at 88 bytes per ns, A at 24, the share of one compute unit when all of them stream),
// and with more than one range the partial sums, written and read at 2.5 TB/s, and 5 us for whoever adds them.  The rates were fitted
// when loads went out in one burst per step; with loads and products alternating the choice is still within 5 % of the fastest of
// all others for 77 of 84 products from 512 x 512 to 8192 x 8192 (l = 64, 96, 128) and within 10 % for 83 (3072 x 3072, l = 64, X A: 19.9
// against 15.5 us with four ranges).
ColumnSplit column_gemm_split(int l, int64_t big, int64_t K) {
  const int64_t ns = (K + COL_BK - 1) / COL_BK;
  ColumnSplit best{1, 1};
  double least = 1e300;
  for (int nt = 4; nt >= 1; nt /= 2)
    for (int ranges : {1, 2, 3, 4, 6, 8}) {
      if (ranges > 1 && ns / ranges < 4) break;               // a step for every wavefront
      const int64_t per = (ns + ranges - 1) / ranges;
      const double wgs = (double)((big + 63) / 64 * (4 / nt)) * (double)ranges;
      const double us = std::ceil(wgs / 256.0) * (double)per * (4.0 * COL_BK) * (l / 88e3 + 16.0 * nt / 24e3) +
                        (ranges > 1 ? 5.0 + (double)ranges * l * (double)big * 8.0 / 2.5e6 : 0.0);
      if (us < least) { least = us; best.nt = nt; best.ranges = ranges; }
    }
  return best;
}

int launch_column_gemm(int mode, int l, int64_t big, int64_t K, const uint16_t* X, const float* A, int64_t lda, ColumnSplit split,
                       float* C, int64_t ldc, uint16_t* packed, float* part, hipStream_t st) {
  if (!column_gemm_supported(l) || big < 1 || K < 1 || lda % 4 || split.ranges < 1 || split.ranges > 8 ||
      (split.nt != 1 && split.nt != 2 && split.nt != 4) || (split.ranges > 1 && !part))
    return LQ_ERR_ARG;
  if (mode == MODE_NT ? K % 4 != 0 : (big % 4 != 0 || big < 4)) return LQ_ERR_ARG;
  // lane offsets into A are 32-bit byte offsets
  if ((mode == MODE_NT ? (uint64_t)big * (uint64_t)lda : (uint64_t)16 * lda + (uint64_t)big) * 4 >= (1ull << 32)) return LQ_ERR_SHAPE;
  ColArgs g;
  g.X = reinterpret_cast<const uintx4*>(X); g.A = A; g.lda = lda; g.big = big; g.K = K;
  g.ns = (int)((K + COL_BK - 1) / COL_BK);
  g.per_range = (g.ns + split.ranges - 1) / split.ranges;
  g.ranges = split.ranges;
  g.ldp = (big + 63) / 64 * 64;
  g.part = part; g.C = C; g.ldc = ldc; g.packed = reinterpret_cast<uintx2*>(packed);
  const int64_t tiles = g.ldp / (16 * split.nt);
  if (tiles * g.ranges >= (1ll << 31)) return LQ_ERR_SHAPE;
  prof::Scope ps(prof::COLUMN_GEMM_BASE + mode * 4 + (l / 32 - 1), st, 2.0 * l * (double)big * (double)K);
  return mode == MODE_NT ? launch_rows<MODE_NT>(g, l, split.nt, tiles, st) : launch_rows<MODE_NN>(g, l, split.nt, tiles, st);
}

}  // namespace lq
