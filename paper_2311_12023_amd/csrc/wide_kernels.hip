// Products between the l x l matrices of the randomized SVD and its wide bases (l rows, thousands of columns): the Gram
// matrix X X^T and the rotation U X.
#include <algorithm>

#include "kernels.h"
#include "profiler.h"

namespace lq {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------------
// Rotation C = U A of up to two wide matrices (the bases Y and B of a Rayleigh-Ritz step share U), on
// v_mfma_f32_32x32x2_f32.  A wavefront owns one 32 x 32 tile of the result and the whole reduction (l <= 128), a workgroup
// the l / 32 tiles of a column block, which share the block of A through L1.  Tiles this small because the operands are
// in cache and a single problem has few of them: 4096 columns at l = 128 are 512 wavefronts, where the streaming GEMM's
// 256-column tiles leave 16 workgroups (one problem, 4096 columns: l = 128 22.9 -> 6.0 us, l = 96 15.4 -> 5.3 us, l = 32
// 5.4 -> 2.9 us).
// The reduction index is permuted (lane half h, sub-chunk c, element e <-> k = 8c + 4h + e) so that U is read with
// 128-bit loads.  LOWER: U is lower triangular and a row tile stops at its diagonal block.
struct RotateArgs {
  const float* U;
  size_t strideU;
  const float* A[2];
  float* C[2];
  int64_t ld[2];                // leading dimension of A and C, a multiple of 32; all of it is multiplied
  size_t stride[2];
  int blocks0;                  // column blocks of the first matrix
};

template <int LT, bool LOWER>
__global__ __launch_bounds__(64 * LT) void rotate_kernel(RotateArgs g) {
  constexpr int l = 32 * LT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, lh = lane >> 5;
  const int seg = (int)blockIdx.x >= g.blocks0, z = blockIdx.y;
  const int64_t ld = g.ld[seg], col = (int64_t)((int)blockIdx.x - (seg ? g.blocks0 : 0)) * 32 + ln;
  const float* __restrict__ A = g.A[seg] + (size_t)z * g.stride[seg] + 4 * lh * ld + col;
  const float* __restrict__ U = g.U + (size_t)z * g.strideU + (32 * w + ln) * l + 4 * lh;
  const int groups = LOWER ? w + 1 : LT;        // of four chunks
  floatx16 acc = {};
  floatx4 u[2][4], a[2][4];
  auto fetch = [&](int q, floatx4 (&ub)[4], floatx4 (&ab)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      ub[c] = *reinterpret_cast<const floatx4*>(U + 32 * q + 8 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) ab[c][e] = A[(int64_t)(32 * q + 8 * c + e) * ld];
    }
  };
  fetch(0, u[0], a[0]);
#pragma unroll
  for (int q = 0; q < LT; ++q) {
    if (q >= groups) break;
    if (q + 1 < groups) fetch(q + 1, u[(q + 1) & 1], a[(q + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);          // the next group's loads are issued before this group's products
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u[q & 1][c][e], a[q & 1][c][e], acc, 0, 0, 0);
  }
  float* __restrict__ C = g.C[seg] + (size_t)z * g.stride[seg] + (int64_t)(32 * w + 4 * lh) * ld + col;
#pragma unroll
  for (int e = 0; e < 16; ++e) C[(int64_t)(8 * (e >> 2) + (e & 3)) * ld] = acc[e];
}

bool rotate_supported(int l) { return l % 32 == 0 && l >= 32 && l <= 128; }

int launch_rotate(int l, const float* U, size_t strideU, bool lower, const float* A0, float* C0, int64_t ld0, size_t stride0,
                  const float* A1, float* C1, int64_t ld1, size_t stride1, int batch, hipStream_t st) {
  if (!rotate_supported(l) || ld0 < 32 || ld0 % 32 || (A1 && (ld1 < 32 || ld1 % 32)) || batch < 1 || batch > 65535) return LQ_ERR_ARG;
  if (ld0 / 32 + (A1 ? ld1 / 32 : 0) >= (1ll << 31)) return LQ_ERR_SHAPE;
  RotateArgs g;
  g.U = U; g.strideU = strideU;
  g.A[0] = A0; g.C[0] = C0; g.ld[0] = ld0; g.stride[0] = stride0;
  g.A[1] = A1; g.C[1] = C1; g.ld[1] = ld1; g.stride[1] = stride1;
  g.blocks0 = (int)(ld0 / 32);
  const dim3 grid((unsigned)(g.blocks0 + (A1 ? ld1 / 32 : 0)), (unsigned)batch);
  prof::Scope ps(prof::ROTATE, st, 8.0 * l * (double)(ld0 + (A1 ? ld1 : 0)) * batch);
#define LQ_ROTATE(LT)                                                                               \
  case LT:                                                                                          \
    if (lower) hipLaunchKernelGGL((rotate_kernel<LT, true>), grid, dim3(64 * LT), 0, st, g);        \
    else hipLaunchKernelGGL((rotate_kernel<LT, false>), grid, dim3(64 * LT), 0, st, g);             \
    break;
  switch (l / 32) { LQ_ROTATE(1) LQ_ROTATE(2) LQ_ROTATE(3) LQ_ROTATE(4) }
#undef LQ_ROTATE
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// ------------------------------------------------------------------------------------------------
// Gram matrix G = X X^T of a wide fp32 matrix in fp64 (the Gram matrix of a basis whose singular values span two decades
// loses what the SVD tolerance needs if it is accumulated in fp32), on v_mfma_f64_16x16x4_f64.  The columns are cut into
// chunks; a chunk of a problem takes l / 32 wavefronts (four to a workgroup), wavefront w owning the 16-row tiles w and
// l/16 - 1 - w of the lower triangle, so that all have l/16 + 1 tile products per 16 columns.  Each lane reads four
// consecutive columns of a row (a permutation of the reduction index that both operands share).  Against fp64 FMAs with
// both operands in LDS (whose reads and conversions bound it: four of each per four products) the operands are converted
// once per l/16 + 1 products and nothing goes through LDS; and the chunks follow the
// batch, where 16 of them left most of the chip idle for a single problem (one problem, l = 128 x 4096: 20.4 -> 7.4 us,
// l = 96 x 11008: 30.9 -> 7.1 us).
// Tiles are stored as they lie in the registers: [problem][chunk][tile pair][4 register][64 lane].
constexpr int gram_waves(int nt) { return nt / 2 < 4 ? nt / 2 : 4; }   // more would halve the registers of each

// One wavefront's part, W = its index: a compile-time constant, since branches around single products (a run-time w) were
// several times slower.
template <int NT, int W>                       // NT = l / 16 row tiles
__device__ __forceinline__ void gram_tiles(const float* __restrict__ Xl, int64_t m, int64_t ldx, int g0, int g1, int lane,
                                           double* __restrict__ P) {
  constexpr int HI = NT - 1 - W;               // the longer row of tiles
  doublex4 lo_acc[W + 1], hi_acc[HI + 1];
#pragma unroll
  for (int t = 0; t <= W; ++t) lo_acc[t] = doublex4{0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t <= HI; ++t) hi_acc[t] = doublex4{0, 0, 0, 0};
  floatx4 ring[2][HI + 1];
  auto fetch = [&](int grp, floatx4 (&x)[HI + 1]) {
#pragma unroll
    for (int t = 0; t <= HI; ++t) x[t] = *reinterpret_cast<const floatx4*>(Xl + (int64_t)16 * t * ldx + (int64_t)16 * grp);
  };
  auto multiply = [&](const floatx4 (&x)[HI + 1]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double v[HI + 1];
#pragma unroll
      for (int t = 0; t <= HI; ++t) v[t] = (double)x[t][e];
#pragma unroll
      for (int t = 0; t <= HI; ++t) {
        hi_acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[HI], v[t], hi_acc[t], 0, 0, 0);
        if (t <= W) lo_acc[t <= W ? t : 0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[W], v[t], lo_acc[t <= W ? t : 0], 0, 0, 0);
      }
    }
  };
  const bool ragged = g1 > g0 && 16 * (int64_t)g1 > m;
  const int gfull = ragged ? g1 - 1 : g1;
  if (g0 < gfull) fetch(g0, ring[0]);
  for (int grp = g0; grp < gfull; grp += 2) {  // prefetches past the end re-read the last group
    fetch(grp + 1 < gfull ? grp + 1 : gfull - 1, ring[1]);
    __builtin_amdgcn_sched_barrier(0);
    multiply(ring[0]);
    if (grp + 1 >= gfull) break;
    fetch(grp + 2 < gfull ? grp + 2 : gfull - 1, ring[0]);
    __builtin_amdgcn_sched_barrier(0);
    multiply(ring[1]);
  }
  if (ragged) {                                // columns past m count as zero whatever the padding holds
    fetch(g1 - 1, ring[0]);
#pragma unroll
    for (int t = 0; t <= HI; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        ring[0][t][e] = 16 * (int64_t)(g1 - 1) + 4 * (lane >> 4) + e < m ? ring[0][t][e] : 0.0f;
    multiply(ring[0]);
  }
#pragma unroll
  for (int t = 0; t <= HI; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      P[(size_t)(HI * (HI + 1) / 2 + t) * 256 + r * 64] = hi_acc[t][r];
      if (t <= W) P[(size_t)(W * (W + 1) / 2 + t) * 256 + r * 64] = lo_acc[t <= W ? t : 0][r];
    }
}

template <int NT>
__global__ __launch_bounds__(64 * gram_waves(NT)) void gram_partial_kernel(const float* __restrict__ X, int64_t m, int64_t ldx,
                                                                           size_t strideX, int groups_per_chunk,
                                                                           double* __restrict__ part) {
  const int w = blockIdx.z * gram_waves(NT) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int chunk = blockIdx.x, z = blockIdx.y;
  const float* __restrict__ Xl = X + (size_t)z * strideX + (int64_t)(lane & 15) * ldx + 4 * (lane >> 4);
  const int g0 = chunk * groups_per_chunk;
  const int gm = (int)((m + 15) / 16);
  const int g1 = g0 + groups_per_chunk < gm ? g0 + groups_per_chunk : gm;
  double* P = part + ((size_t)z * gridDim.x + chunk) * (NT * (NT + 1) / 2 * 256) + lane;
#define LQ_GRAM_WAVE(W) \
  if constexpr (W < NT / 2) { if (w == W) gram_tiles<NT, W>(Xl, m, ldx, g0, g1, lane, P); }
  LQ_GRAM_WAVE(0) LQ_GRAM_WAVE(1) LQ_GRAM_WAVE(2) LQ_GRAM_WAVE(3)
  LQ_GRAM_WAVE(4) LQ_GRAM_WAVE(5) LQ_GRAM_WAVE(6) LQ_GRAM_WAVE(7)
#undef LQ_GRAM_WAVE
}

// G = sum of the chunks, the tiles above the diagonal mirrored.  One workgroup per accumulator register of a tile pair and
// problem; register r of a lane is row 4 r + lane / 16, column lane % 16.  Bound by memory round trips: each of the up to
// eight wavefronts adds a contiguous range of the chunks, GRAM_REDUCE_DEPTH in flight at a time, and the ranges are added in
// order through LDS (one problem of 4096 columns, l = 128: 6.8 -> 4.5 us against one thread for all chunks of an element, l = 32:
// 4.6 -> 3.3).
constexpr int GRAM_REDUCE_DEPTH = 16, GRAM_REDUCE_WAVES = 8;
__global__ __launch_bounds__(64 * GRAM_REDUCE_WAVES) void gram_reduce_kernel(const double* __restrict__ part, double* __restrict__ G,
                                                                             int l, int chunks, int per_wave) {
  __shared__ double s_sum[GRAM_REDUCE_WAVES][64];
  const int pair = blockIdx.x >> 2, r = blockIdx.x & 3, pairs = gridDim.x >> 2, z = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  int ti = 0, tj = pair;
  while (tj > ti) { tj -= ti + 1; ++ti; }
  const size_t pitch = (size_t)pairs * 256;
  const double* P = part + ((size_t)z * chunks * pairs + pair) * 256 + 64 * r + lane;
  const int c1 = (wave + 1) * per_wave < chunks ? (wave + 1) * per_wave : chunks;
  double s = 0.0;
  for (int c = wave * per_wave; c < c1; c += GRAM_REDUCE_DEPTH) {
    double v[GRAM_REDUCE_DEPTH];
#pragma unroll
    for (int u = 0; u < GRAM_REDUCE_DEPTH; ++u) v[u] = P[(size_t)(c + u < c1 ? c + u : c1 - 1) * pitch];
#pragma unroll
    for (int u = 0; u < GRAM_REDUCE_DEPTH; ++u) s += c + u < c1 ? v[u] : 0.0;
  }
  if (waves > 1) {
    s_sum[wave][lane] = s;
    __syncthreads();
    if (wave > 0) return;
    for (int w = 1; w < waves; ++w) s += s_sum[w][lane];
  }
  const int i = 16 * ti + 4 * r + (lane >> 4), j = 16 * tj + (lane & 15);
  double* Gz = G + (size_t)z * l * l;
  Gz[(size_t)i * l + j] = s;
  if (ti != tj) Gz[(size_t)j * l + i] = s;
}

template <int NT>
static void launch_gram_partial(const float* X, int64_t m, int64_t ldx, size_t strideX, int chunks, int gpc, double* part,
                                int batch, hipStream_t st) {
  hipLaunchKernelGGL(gram_partial_kernel<NT>, dim3(chunks, batch, (NT / 2 + gram_waves(NT) - 1) / gram_waves(NT)),
                     dim3(64 * gram_waves(NT)), 0, st, X, m, ldx, strideX, gpc, part);
}

int launch_gram(const float* X, int l, int64_t m, int64_t ldx, size_t strideX, double* part, size_t part_doubles, double* G,
                int batch, hipStream_t st) {
  if (l % 32 || l < 32 || l > 256 || m < 1 || ldx % 4 || ldx < (m + 15) / 16 * 16 || m > (1ll << 34) || batch < 1 || batch > 65535)
    return LQ_ERR_ARG;
  const int nt = l / 16, pairs = nt * (nt + 1) / 2;
  const int64_t groups = (m + 15) / 16;
  // Enough chunks for about two wavefronts per SIMD, no chunk shorter than two groups, no more partial results than the
  // scratch holds.
  int64_t chunks = (2048 + (int64_t)batch * nt / 2 - 1) / ((int64_t)batch * nt / 2);
  chunks = std::min<int64_t>(chunks, GRAM_CHUNKS_MAX);
  chunks = std::min<int64_t>(chunks, (groups + 1) / 2);
  chunks = std::min<int64_t>(chunks, (int64_t)(part_doubles / ((size_t)batch * pairs * 256)));
  if (chunks < 1) return LQ_ERR_ARG;
  const int gpc = (int)((groups + chunks - 1) / chunks);
  chunks = (groups + gpc - 1) / gpc;
  prof::Scope ps(prof::GRAM, st, (double)l * m * 4.0 * batch);
  switch (nt) {
    case 2: launch_gram_partial<2>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 4: launch_gram_partial<4>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 6: launch_gram_partial<6>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 8: launch_gram_partial<8>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 10: launch_gram_partial<10>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 12: launch_gram_partial<12>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 14: launch_gram_partial<14>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    case 16: launch_gram_partial<16>(X, m, ldx, strideX, (int)chunks, gpc, part, batch, st); break;
    default: return LQ_ERR_ARG;
  }
  LQ_HIP_TRY(hipGetLastError());
  const int waves = (int)std::min<int64_t>(GRAM_REDUCE_WAVES, (chunks + GRAM_REDUCE_DEPTH - 1) / GRAM_REDUCE_DEPTH);
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(4 * pairs, batch), dim3(64 * waves), 0, st, (const double*)part, G, l, (int)chunks,
                     ((int)chunks + waves - 1) / waves);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

}  // namespace lq
