// Small dense kernels of the randomized SVD: Cholesky factors for the orthonormalisation, the filter steps of the cold
// start, a parallel Jacobi eigen-solver for blocks of more than 128 rows (eig_kernels.hip has the others), row norms, sketch
// generation and factor assembly (Algorithm 4), Fisher weights.  They are latency-, not throughput-critical; the
// factors and the solver keep their working set in registers or LDS where it fits.
#include <cmath>

#include "dense_device.h"
#include "kernels.h"
#include "mfma_device.h"
#include "profiler.h"

namespace lq {

// ------------------------------------------------------------------------------------------------
// Cholesky, right-looking, one workgroup per problem.  PACKED: the lower triangle is worked on in LDS
// (row-packed); otherwise in place in global memory.
template <bool PACKED>
__global__ __launch_bounds__(256) void cholesky_kernel(double* __restrict__ Gall, int l) {
  extern __shared__ double lds[];
  __shared__ double s_inv;
  double* G = Gall + (size_t)blockIdx.x * l * l;
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  double* Lw = PACKED ? lds : G;
  auto at = [&](int i, int j) -> double& { return PACKED ? Lw[(size_t)i * (i + 1) / 2 + j] : Lw[(size_t)i * l + j]; };
  if (PACKED) {
    for (int idx = tid; idx < l * l; idx += 256) {
      const int i = idx / l, j = idx % l;
      if (j <= i) at(i, j) = G[idx];
    }
  }
  // A pivot is compared with the row's own squared norm (what is left of row j after the rows before it have been
  // taken out is negligible below 1e-6 of its length), not with the largest one: the rows of a block may differ in
  // length by many orders of magnitude (filtered rows beside rows kept at unit length).
  __shared__ double s_diag[256];
  for (int i = tid; i < l; i += 256) s_diag[i] = G[(size_t)i * l + i];
  for (int j = 0; j < l; ++j) {
    __syncthreads();
    const double piv = at(j, j);
    const bool ok = piv > 1e-12 * s_diag[j];
    const double cjj = ok ? sqrt(piv) : 0.0;
    const double inv = ok ? 1.0 / cjj : 0.0;
    for (int i = j + 1 + tid; i < l; i += 256) at(i, j) *= inv;
    __syncthreads();
    if (tid == 0) at(j, j) = cjj;
    for (int i = j + 1 + ty; i < l; i += 16) {
      const double cij = at(i, j);
      for (int kk = j + 1 + tx; kk <= i; kk += 16) at(i, kk) -= cij * at(kk, j);
    }
  }
  __syncthreads();
  if (PACKED) {
    for (int idx = tid; idx < l * l; idx += 256) {
      const int i = idx / l, j = idx % l;
      if (j <= i) G[idx] = at(i, j);
    }
  }
  (void)s_inv;
}

static size_t g_max_lds = 0;
static size_t max_lds_bytes() {
  if (g_max_lds == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 0)
      g_max_lds = (size_t)v;
    else
      g_max_lds = 65536;
  }
  return g_max_lds;
}
size_t lds_limit_for_tests() { return max_lds_bytes(); }

int launch_cholesky(double* G, int l, int batch, hipStream_t st) {
  const size_t need = (size_t)l * (l + 1) / 2 * sizeof(double);
  prof::Scope ps(prof::CHOLESKY, st, (double)l * l * 8.0 * batch);
  if (need + 64 <= 65536 && need + 64 <= max_lds_bytes())
    hipLaunchKernelGGL(cholesky_kernel<true>, dim3(batch), dim3(256), need, st, G, l);
  else
    hipLaunchKernelGGL(cholesky_kernel<false>, dim3(batch), dim3(256), 0, st, G, l);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// ------------------------------------------------------------------------------------------------
// Forward substitution X <- C^-1 X, one lane per column of X, the column kept in LDS.
__global__ __launch_bounds__(64) void trsm_kernel(const double* __restrict__ Call, int l, float* __restrict__ Xall,
                                                  int64_t m, int64_t ldx, size_t strideX) {
  extern __shared__ float ys[];   // [l][64]
  const int z = blockIdx.y, lane = threadIdx.x;
  const double* __restrict__ Cf = Call + (size_t)z * l * l;
  float* X = Xall + (size_t)z * strideX;
  const int64_t col = (int64_t)blockIdx.x * 64 + lane;
  const bool live = col < m;
  for (int i = 0; i < l; ++i) {
    float acc = live ? X[(size_t)i * ldx + col] : 0.0f;
    const double* __restrict__ crow = Cf + (size_t)i * l;
    for (int kk = 0; kk < i; ++kk) acc = fmaf(-(float)crow[kk], ys[kk * 64 + lane], acc);
    const double cii = crow[i];
    const float y = cii > 0.0 ? acc / (float)cii : 0.0f;
    ys[i * 64 + lane] = y;
    if (live) X[(size_t)i * ldx + col] = y;
  }
}

int launch_trsm(const double* Cfac, int l, float* X, int64_t m, int64_t ldx, size_t strideX, int batch,
                hipStream_t st) {
  prof::Scope ps(prof::TRSM, st, (double)l * m * 8.0 * batch);
  hipLaunchKernelGGL(trsm_kernel, dim3((unsigned)((m + 63) / 64), batch), dim3(64), (size_t)l * 64 * sizeof(float), st,
                     Cfac, l, X, m, ldx, strideX);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// ------------------------------------------------------------------------------------------------
// Symmetric eigen-decomposition, two-sided Jacobi with a round-robin ordering: every round applies
// l/2 disjoint rotations at once, M <- J^T M J as independent 2x2 blocks, Vt <- J^T Vt as row pairs.
constexpr int JT = 512;

// STORE: 0 = M and Vt in global memory, 1 = M in LDS, 2 = M and Vt in LDS.
template <int STORE>
__global__ __launch_bounds__(JT) void jacobi_eig_kernel(double* __restrict__ Gall, int l, double* __restrict__ Vall,
                                                        float* __restrict__ Utall, double* __restrict__ lamall) {
  extern __shared__ double lds[];
  __shared__ double s_c[128], s_s[128];
  __shared__ int s_p[128], s_q[128];
  __shared__ int s_rot;
  __shared__ int s_rank[256];
  const int z = blockIdx.x, tid = threadIdx.x;
  double* G = Gall + (size_t)z * l * l;
  const int pm = STORE >= 1 ? l + 1 : l;       // row pitch of M
  const int pv = STORE == 2 ? l + 1 : l;       // row pitch of Vt
  double* M = STORE >= 1 ? lds : G;
  double* Vt = STORE == 2 ? lds + (size_t)l * (l + 1) : Vall + (size_t)z * l * l;
  const int ll = l * l, half = l / 2;
  for (int idx = tid; idx < ll; idx += JT) {
    const int r = idx / l, cidx = idx % l;
    if (STORE >= 1) M[r * pm + cidx] = G[idx];
    Vt[r * pv + cidx] = (r == cidx) ? 1.0 : 0.0;
  }
  __syncthreads();
  for (int sweep = 0; sweep < 40; ++sweep) {
    if (tid == 0) s_rot = 0;
    __syncthreads();
    for (int round = 0; round < l - 1; ++round) {
      if (tid < half) {
        int p, q;
        circle_pair(tid, round, l, p, q);
        const double mpp = M[p * pm + p], mqq = M[q * pm + q], mpq = M[p * pm + q];
        double c = 1.0, s = 0.0;
        if (mpq != 0.0 && fabs(mpq) > 1e-10 * sqrt(fabs(mpp * mqq))) {
          const double tau = (mqq - mpp) / (2.0 * mpq);
          const double t = (tau >= 0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
          c = 1.0 / sqrt(1.0 + t * t);
          s = t * c;
          s_rot = 1;
        }
        s_c[tid] = c; s_s[tid] = s; s_p[tid] = p; s_q[tid] = q;
      }
      __syncthreads();
      // M <- J^T M J on the blocks a <= b (rows of pair a, columns of pair b); the mirror block is written too
      for (int blk = tid; blk < half * half; blk += JT) {
        const int a = blk / half, b = blk % half;
        if (b < a) continue;
        const double c1 = s_c[a], s1 = s_s[a], c2 = s_c[b], s2 = s_s[b];
        if (s1 == 0.0 && s2 == 0.0) continue;
        const int p = s_p[a], q = s_q[a], p2 = s_p[b], q2 = s_q[b];
        const double m00 = M[p * pm + p2], m01 = M[p * pm + q2];
        const double m10 = M[q * pm + p2], m11 = M[q * pm + q2];
        const double r00 = c1 * m00 - s1 * m10, r01 = c1 * m01 - s1 * m11;   // rows: J^T from the left
        const double r10 = s1 * m00 + c1 * m10, r11 = s1 * m01 + c1 * m11;
        const double n00 = c2 * r00 - s2 * r01, n01 = s2 * r00 + c2 * r01;
        const double n10 = c2 * r10 - s2 * r11, n11 = s2 * r10 + c2 * r11;
        M[p * pm + p2] = n00; M[p * pm + q2] = n01; M[q * pm + p2] = n10; M[q * pm + q2] = n11;
        if (a != b) { M[p2 * pm + p] = n00; M[q2 * pm + p] = n01; M[p2 * pm + q] = n10; M[q2 * pm + q] = n11; }
      }
      // Vt <- J^T Vt
      for (int it = tid; it < half * l; it += JT) {
        const int a = it / l, col = it % l;
        const double c1 = s_c[a], s1 = s_s[a];
        if (s1 == 0.0) continue;
        const int p = s_p[a], q = s_q[a];
        const double vp = Vt[p * pv + col], vq = Vt[q * pv + col];
        Vt[p * pv + col] = c1 * vp - s1 * vq;
        Vt[q * pv + col] = s1 * vp + c1 * vq;
      }
      __syncthreads();
    }
    if (s_rot == 0) break;   // every thread reads the flag after the round's closing barrier
    __syncthreads();
  }
  // descending sort by rank counting, then emit fp32 eigenvectors as rows
  for (int i = tid; i < l; i += JT) {
    const double li = M[i * pm + i];
    int r = 0;
    for (int j = 0; j < l; ++j) r += sorts_before(M[j * pm + j], j, li, i) ? 1 : 0;
    s_rank[i] = r;
    lamall[(size_t)z * l + r] = li > 0.0 ? li : 0.0;
  }
  __syncthreads();
  float* Ut = Utall + (size_t)z * l * l;
  for (int idx = tid; idx < ll; idx += JT) {
    const int i = idx / l, col = idx % l;
    Ut[(size_t)s_rank[i] * l + col] = (float)Vt[i * pv + col];
  }
}

// lam[z][i] = sum_j X[z][i][j]^2 in fp64: the Ritz values sigma_i^2 as the squared row norms of the rotated
// projected matrix.
__global__ __launch_bounds__(256) void row_sumsq_kernel(const float* __restrict__ X, int64_t m, int64_t ldx,
                                                        size_t strideX, int l, double* __restrict__ lam) {
  __shared__ double s_sum[4];
  const int row = blockIdx.x, z = blockIdx.y, tid = threadIdx.x;
  const float* x = X + (size_t)z * strideX + (size_t)row * ldx;
  double s = 0.0;
  const int64_t quads = m / 4;                 // rows start on 16-byte boundaries
#pragma unroll 4
  for (int64_t j = tid; j < quads; j += 256) {
    const float4 v = reinterpret_cast<const float4*>(x)[j];
    s = fma((double)v.x, (double)v.x, s); s = fma((double)v.y, (double)v.y, s);
    s = fma((double)v.z, (double)v.z, s); s = fma((double)v.w, (double)v.w, s);
  }
  if (tid < m - 4 * quads) { const double v = x[4 * quads + tid]; s = fma(v, v, s); }
  for (int off = 1; off < 64; off <<= 1) s += __shfl_xor(s, off);
  if ((tid & 63) == 0) s_sum[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) lam[(size_t)z * l + row] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

// res[i] = |G_i - lam[i] Y_i|^2 for the first `rows` rows: squared residual norms of the Ritz pairs (lam_i, Y_i) of the
// operator that G = Y M was formed with.
__global__ __launch_bounds__(256) void ritz_residual_kernel(const float* __restrict__ G, const float* __restrict__ Y,
                                                            const double* __restrict__ lam, int64_t m, int64_t ldx,
                                                            double* __restrict__ res) {
  __shared__ double s_sum[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const float* g = G + (size_t)row * ldx;
  const float* y = Y + (size_t)row * ldx;
  const double th = lam[row];
  double s = 0.0;
  for (int64_t j = tid; j < m; j += 256) { const double v = (double)g[j] - th * (double)y[j]; s = fma(v, v, s); }
  for (int off = 1; off < 64; off <<= 1) s += __shfl_xor(s, off);
  if ((tid & 63) == 0) s_sum[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) res[row] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

int launch_ritz_residual(const float* G, const float* Y, const double* lam, int rows, int64_t m, int64_t ldx, double* res,
                         hipStream_t st) {
  prof::Scope ps(prof::MISC, st, (double)rows * m * 8.0);
  hipLaunchKernelGGL(ritz_residual_kernel, dim3(rows), dim3(256), 0, st, G, Y, lam, m, ldx, res);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

int launch_row_sumsq(const float* X, int l, int64_t m, int64_t ldx, size_t strideX, double* lam, int batch,
                     hipStream_t st) {
  prof::Scope ps(prof::MISC, st, (double)l * m * 4.0 * batch);
  hipLaunchKernelGGL(row_sumsq_kernel, dim3(l, batch), dim3(256), 0, st, X, m, ldx, strideX, l, lam);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

int launch_jacobi_eig(double* G, int l, double* vt, float* Ut, double* lambda, int batch, hipStream_t st) {
  if (l > 256 || l % 2) return LQ_ERR_ARG;
  const size_t lim = max_lds_bytes() - 8192;          // static arrays of the kernel
  const size_t one = (size_t)l * (l + 1) * sizeof(double);
  static LdsLimit limit1, limit2;
  LQ_TRY(limit1.raise(reinterpret_cast<const void*>(jacobi_eig_kernel<1>), lim));
  LQ_TRY(limit2.raise(reinterpret_cast<const void*>(jacobi_eig_kernel<2>), lim));
  prof::Scope ps(prof::JACOBI, st, (double)l * l * 8.0 * batch);
  if (2 * one <= lim)
    hipLaunchKernelGGL(jacobi_eig_kernel<2>, dim3(batch), dim3(JT), 2 * one, st, G, l, vt, Ut, lambda);
  else if (one <= lim)
    hipLaunchKernelGGL(jacobi_eig_kernel<1>, dim3(batch), dim3(JT), one, st, G, l, vt, Ut, lambda);
  else
    hipLaunchKernelGGL(jacobi_eig_kernel<0>, dim3(batch), dim3(JT), 0, st, G, l, vt, Ut, lambda);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// ------------------------------------------------------------------------------------------------
__device__ inline uint64_t mix64(uint64_t x) {
  x += 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

__global__ __launch_bounds__(256) void gaussian_fill_kernel(float* __restrict__ X, int l, int64_t m, int64_t ldx,
                                                            uint64_t seed) {
  const int64_t total = (int64_t)l * ldx;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int64_t row = idx / ldx, col = idx % ldx;
    float val = 0.0f;
    if (col < m) {
      const uint64_t h = mix64(mix64(seed) ^ (uint64_t)(row * m + col));
      const float u1 = ((float)(uint32_t)(h >> 40) + 0.5f) * (1.0f / 16777216.0f);   // (0,1)
      const float u2 = ((float)(uint32_t)((h >> 8) & 0xffffffu)) * (1.0f / 16777216.0f);
      val = sqrtf(-2.0f * logf(u1)) * cosf(6.28318530717958647692f * u2);
    }
    X[idx] = val;
  }
}

// Largest finite |x[i]|: 1024 workgroups leave their maxima in out[0..1023], then one workgroup reduces them into
// out[1024] (two launches; a maximum does not depend on the order it is taken in).
__global__ __launch_bounds__(256) void absmax_kernel(const float* __restrict__ x, int64_t n, float* __restrict__ out,
                                                     int stage) {
  __shared__ float s_max[256];
  const int tid = threadIdx.x;
  float m = 0.0f;
  if (stage == 0) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < n; i += (int64_t)gridDim.x * 256) {
      const float a = fabsf(x[i]);
      if (a < __builtin_inff()) m = fmaxf(m, a);     // false for NaN as well
    }
  } else {
    for (int i = tid; i < 1024; i += 256) m = fmaxf(m, out[i]);
  }
  s_max[tid] = m;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (tid < w) s_max[tid] = fmaxf(s_max[tid], s_max[tid + w]);
    __syncthreads();
  }
  if (tid == 0) out[stage == 0 ? blockIdx.x : 1024] = s_max[0];
}

int launch_absmax(const float* x, int64_t n, float* out, hipStream_t st) {
  prof::Scope ps(prof::ABSMAX, st, (double)n * 4.0);
  hipLaunchKernelGGL(absmax_kernel, dim3(1024), dim3(256), 0, st, x, n, out, 0);
  LQ_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(absmax_kernel, dim3(1), dim3(256), 0, st, x, n, out, 1);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// Rows of X against the first `locked` rows of L (orthonormal): rows i >= locked lose their components along them,
// x_i <- x_i - sum_o (x_i . l_o) l_o; rows i < locked become copies of l_i.  One workgroup per row; inner products in
// fp32 with a fixed summation order.  locked <= DEFLATE_MAX.
constexpr int DEFLATE_MAX = 16;

__global__ __launch_bounds__(256) void deflate_rows_kernel(float* __restrict__ X, const float* __restrict__ L, int locked,
                                                           int64_t m4, int64_t ldx) {
  __shared__ float s_part[4][DEFLATE_MAX];
  __shared__ float s_dot[DEFLATE_MAX];
  const int row = blockIdx.x, tid = threadIdx.x;
  float4* x = reinterpret_cast<float4*>(X + (size_t)row * ldx);
  if (row < locked) {
    const float4* src = reinterpret_cast<const float4*>(L + (size_t)row * ldx);
    for (int64_t j = tid; j < m4; j += 256) x[j] = src[j];
    return;
  }
  float dot[DEFLATE_MAX];
#pragma unroll
  for (int o = 0; o < DEFLATE_MAX; ++o) dot[o] = 0.f;
  for (int64_t j = tid; j < m4; j += 256) {
    const float4 v = x[j];
#pragma unroll
    for (int o = 0; o < DEFLATE_MAX; ++o)
      if (o < locked) {
        const float4 u = reinterpret_cast<const float4*>(L + (size_t)o * ldx)[j];
        dot[o] = fmaf(v.x, u.x, fmaf(v.y, u.y, fmaf(v.z, u.z, fmaf(v.w, u.w, dot[o]))));
      }
  }
#pragma unroll
  for (int o = 0; o < DEFLATE_MAX; ++o) {
    float t = dot[o];
    for (int off = 1; off < 64; off <<= 1) t += __shfl_xor(t, off);
    if ((tid & 63) == 0) s_part[tid >> 6][o] = t;
  }
  __syncthreads();
  if (tid < DEFLATE_MAX) s_dot[tid] = (s_part[0][tid] + s_part[1][tid]) + (s_part[2][tid] + s_part[3][tid]);
  __syncthreads();
  for (int64_t j = tid; j < m4; j += 256) {
    float4 v = x[j];
#pragma unroll
    for (int o = 0; o < DEFLATE_MAX; ++o)
      if (o < locked) {
        const float4 u = reinterpret_cast<const float4*>(L + (size_t)o * ldx)[j];
        const float c = s_dot[o];
        v.x = fmaf(-c, u.x, v.x); v.y = fmaf(-c, u.y, v.y); v.z = fmaf(-c, u.z, v.z); v.w = fmaf(-c, u.w, v.w);
      }
    x[j] = v;
  }
}

int launch_deflate_rows(float* X, const float* L, int l, int locked, int64_t m, int64_t ldx, hipStream_t st) {
  if (locked < 0 || locked > DEFLATE_MAX || ldx % 4 != 0) return LQ_ERR_ARG;
  if (locked == 0) return LQ_OK;
  prof::Scope ps(prof::MISC, st, (double)l * m * 4.0 * 2.0 * (1 + locked));
  hipLaunchKernelGGL(deflate_rows_kernel, dim3(l), dim3(256), 0, st, X, L, locked, (m + 3) / 4, ldx);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// A filter step.  X is read as it is or as the sum of the ranges that launch_column_gemm left, and the result is also written in
// the operand layout of the next product: neither takes a launch of its own.  An XCD's workgroups have l / 8 neighbouring rows: at
// l = 64 and 128 whole lines of the operand layout (8 rows of 16 bytes) come out of one L2; at l = 32 and 96 some lines are written
// in two parts by two XCDs.
struct FilterArgs {
  float* X; const float* part; int ranges; size_t next;       // part NULL: X itself
  float a, b, c;
  const float* Y; const float* Z; const float* L;
  int locked, q4, row_tiles;
  uintx2* packed;
};

__device__ __forceinline__ float4 filter_combine(const FilterArgs& g, int64_t row, int j) {
  const int64_t at = row * g.q4 + j;
  float4 t;
  if (g.part) {
    const float* p = g.part + 4 * at;
    t = *reinterpret_cast<const float4*>(p);
    for (int r = 1; r < g.ranges; ++r) {
      const float4 u = *reinterpret_cast<const float4*>(p + r * g.next);
      t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
  } else {
    t = reinterpret_cast<const float4*>(g.X)[at];
  }
  if (g.Y) {
    const float4 u = reinterpret_cast<const float4*>(g.Y)[at];
    t.x = fmaf(g.a, t.x, g.b * u.x); t.y = fmaf(g.a, t.y, g.b * u.y); t.z = fmaf(g.a, t.z, g.b * u.z); t.w = fmaf(g.a, t.w, g.b * u.w);
    if (g.Z) {
      const float4 w = reinterpret_cast<const float4*>(g.Z)[at];
      t.x = fmaf(g.c, w.x, t.x); t.y = fmaf(g.c, w.y, t.y); t.z = fmaf(g.c, w.z, t.z); t.w = fmaf(g.c, w.w, t.w);
    }
  }
  return t;
}

__device__ __forceinline__ void filter_store(const FilterArgs& g, int64_t row, int j, float4 t) {
  reinterpret_cast<float4*>(g.X)[row * g.q4 + j] = t;
  if (g.packed) store_packed(g.packed, g.row_tiles, (int)row, 4 * (int64_t)j, floatx4{t.x, t.y, t.z, t.w});
}

// Nothing locked: elementwise.  gridDim = (rows, quads / 256).
__global__ __launch_bounds__(256) void filter_combine_kernel(FilterArgs g) {
  const int64_t row = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int j = blockIdx.y * 256 + threadIdx.x;
  if (j < g.q4) filter_store(g, row, j, filter_combine(g, row, j));
}

// The combination and deflate_rows in one pass over the rows (one workgroup per row, the combined row in registers; 128 rows x
// 4096, four locked: two launches 17.4, this 5.9 us).  RC float4 per thread bound the row length; LB >= locked fixes the register
// arrays.
constexpr int FS_THREADS = 512, FS_RC = 8;

template <int LB>
__global__ __launch_bounds__(FS_THREADS) void filter_step_kernel(FilterArgs g) {
  __shared__ float s_part[FS_THREADS / 64][LB];
  const int tid = threadIdx.x, locked = g.locked, q4 = g.q4;
  const int64_t row = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const float4* l4 = reinterpret_cast<const float4*>(g.L);
  if (row < locked) {
    for (int j = tid; j < q4; j += FS_THREADS) filter_store(g, row, j, l4[row * q4 + j]);
    return;
  }
  float4 v[FS_RC];
  float dot[LB];
#pragma unroll
  for (int o = 0; o < LB; ++o) dot[o] = 0.f;
#pragma unroll
  for (int r = 0; r < FS_RC; ++r) {
    const int j = tid + r * FS_THREADS;
    v[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < q4) {
      const float4 t = filter_combine(g, row, j);
      v[r] = t;
#pragma unroll
      for (int o = 0; o < LB; ++o) {
        const float4 u = l4[(int64_t)(o < locked ? o : 0) * q4 + j];       // past the last one: a row again, its sum unused
        dot[o] = fmaf(t.x, u.x, fmaf(t.y, u.y, fmaf(t.z, u.z, fmaf(t.w, u.w, dot[o]))));
      }
    }
  }
#pragma unroll
  for (int o = 0; o < LB; ++o) {
    float t = dot[o];
    for (int off = 1; off < 64; off <<= 1) t += __shfl_xor(t, off);
    if ((tid & 63) == 0) s_part[tid >> 6][o] = t;
  }
  __syncthreads();
#pragma unroll
  for (int o = 0; o < LB; ++o) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < FS_THREADS / 64; ++w) t += s_part[w][o];
    dot[o] = o < locked ? -t : 0.f;
  }
#pragma unroll
  for (int r = 0; r < FS_RC; ++r) {
    const int j = tid + r * FS_THREADS;
    if (j < q4) {
      float4 t = v[r];
#pragma unroll
      for (int o = 0; o < LB; ++o) {
        const float4 u = l4[(int64_t)(o < locked ? o : 0) * q4 + j];
        t.x = fmaf(dot[o], u.x, t.x); t.y = fmaf(dot[o], u.y, t.y); t.z = fmaf(dot[o], u.z, t.z); t.w = fmaf(dot[o], u.w, t.w);
      }
      filter_store(g, row, j, t);
    }
  }
}

int launch_filter_step(float* X, float a, const float* Y, float b, const float* Z, float c, const float* L, int l, int locked,
                       int64_t m, int64_t ldx, hipStream_t st, const float* part, int ranges, uint16_t* packed) {
  if (l < 8 || l % 8 || locked < 0 || locked > DEFLATE_MAX || ldx % 4 != 0 || ldx > (1ll << 31) || (Z && !Y)) return LQ_ERR_ARG;
  if (packed && (l % 16 || ldx % 64)) return LQ_ERR_ARG;
  const bool whole = locked > 0 && ldx <= (int64_t)4 * FS_THREADS * FS_RC;      // a row fits the registers of a workgroup
  if (locked == 0 && !Y && !part && !packed) return LQ_OK;
  FilterArgs g;
  g.X = X; g.part = part; g.ranges = ranges; g.next = (size_t)l * ldx;
  g.a = a; g.b = b; g.c = c; g.Y = Y; g.Z = Z; g.L = L;
  g.locked = locked; g.q4 = (int)(ldx / 4); g.row_tiles = l / 16;
  g.packed = whole || locked == 0 ? reinterpret_cast<uintx2*>(packed) : nullptr;
  if (whole || locked == 0 || Y || part) {
    prof::Scope ps(prof::MISC, st, (double)l * ldx * 4.0 * (1 + (part ? ranges : 1) + (Y ? 1 : 0) + (Z ? 1 : 0)));
    if (!whole) hipLaunchKernelGGL(filter_combine_kernel, dim3(l, (unsigned)((g.q4 + 255) / 256)), dim3(256), 0, st, g);
    else if (locked <= 4) hipLaunchKernelGGL(filter_step_kernel<4>, dim3(l), dim3(FS_THREADS), 0, st, g);
    else if (locked <= 8) hipLaunchKernelGGL(filter_step_kernel<8>, dim3(l), dim3(FS_THREADS), 0, st, g);
    else hipLaunchKernelGGL(filter_step_kernel<16>, dim3(l), dim3(FS_THREADS), 0, st, g);
    LQ_HIP_TRY(hipGetLastError());
  }
  if (whole || locked == 0) return LQ_OK;
  LQ_TRY(launch_deflate_rows(X, L, l, locked, m, ldx, st));
  return packed ? launch_column_sum(l, X, ldx, 1, ldx, nullptr, 0, packed, st) : LQ_OK;
}

int launch_gaussian_fill(float* X, int l, int64_t m, int64_t ldx, uint64_t seed, hipStream_t st) {
  const int64_t total = (int64_t)l * ldx;
  const int64_t want = (total + 255) / 256;
  hipLaunchKernelGGL(gaussian_fill_kernel, dim3((unsigned)(want < 4096 ? want : 4096)), dim3(256), 0, st, X, l, m, ldx,
                     seed);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

__global__ __launch_bounds__(256) void scale_matrix_kernel(const float* __restrict__ A, int64_t d, int64_t k,
                                                           const float* __restrict__ sr,
                                                           const float* __restrict__ sc, float* __restrict__ out) {
  const int64_t total = d * k;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int64_t i = idx / k, j = idx % k;
    out[idx] = sr[i] * A[idx] * sc[j];
  }
}

int launch_scale_matrix(const float* A, int64_t d, int64_t k, const float* sr, const float* sc, float* out,
                        hipStream_t st) {
  const int64_t want = (d * k + 255) / 256;
  hipLaunchKernelGGL(scale_matrix_kernel, dim3((unsigned)(want < 8192 ? want : 8192)), dim3(256), 0, st, A, d, k,
                     sr, sc, out);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

__global__ void sqrt_vecs_kernel(const float* __restrict__ w, int64_t n, float* __restrict__ s, float* __restrict__ rs) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) {
    const float r = sqrtf(w[i]);
    s[i] = r;
    rs[i] = 1.0f / r;
  }
}

int launch_sqrt_vecs(const float* w, int64_t n, float* s, float* rs, hipStream_t st) {
  hipLaunchKernelGGL(sqrt_vecs_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, n, s, rs);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// L1 (d x rank) and L2 (rank x k) from the Ritz-ordered bases.
__global__ __launch_bounds__(256) void assemble_factors_kernel(const float* __restrict__ Y, int64_t ldy,
                                                               const float* __restrict__ B, int64_t ldb,
                                                               const double* __restrict__ lambda, int rank, int64_t d,
                                                               int64_t k, const float* __restrict__ rsr,
                                                               const float* __restrict__ rsc, float* __restrict__ L1,
                                                               float* __restrict__ L2) {
  const int64_t n1 = d * rank, n2 = (int64_t)rank * k;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < n1 + n2; idx += (int64_t)gridDim.x * 256) {
    if (idx < n1) {
      const int64_t i = idx / rank;
      const int p = (int)(idx % rank);
      const float rs = (float)sqrt(sqrt(lambda[p]));           // sqrt(sigma)
      float val = Y[(size_t)p * ldy + i] * rs;
      if (rsr) val *= rsr[i];
      L1[idx] = val;
    } else {
      const int64_t e = idx - n1;
      const int p = (int)(e / k);
      const int64_t j = e % k;
      const double sg = sqrt(lambda[p]);
      const float inv = sg > 0.0 ? (float)(1.0 / sqrt(sg)) : 0.0f;
      float val = B[(size_t)p * ldb + j] * inv;
      if (rsc) val *= rsc[j];
      L2[e] = val;
    }
  }
}

int launch_assemble_factors(const float* Y, int64_t ldy, const float* B, int64_t ldb, const double* lambda, int rank,
                            int64_t d, int64_t k, const float* rsr, const float* rsc, float* L1, float* L2,
                            hipStream_t st) {
  const int64_t want = ((d + k) * rank + 255) / 256;
  hipLaunchKernelGGL(assemble_factors_kernel, dim3((unsigned)(want < 4096 ? want : 4096)), dim3(256), 0, st, Y, ldy, B,
                     ldb, lambda, rank, d, k, rsr, rsc, L1, L2);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// ---- RowAverage / ColAverage of sqrt(F) (Section 3.3, Algorithm 4) ----------------------------------------------
// Pass 1: a workgroup takes FISHER_ROWS rows; thread t walks the columns t, t + 256, ...: it adds sqrt(F) down its
// column into one partial column sum per workgroup and across into FISHER_ROWS row sums, all in fp64.
constexpr int FISHER_ROWS = 16;

__global__ __launch_bounds__(256) void fisher_partial_kernel(const float* __restrict__ F, int64_t d, int64_t k,
                                                             double* __restrict__ rowsum,
                                                             double* __restrict__ colpart) {
  __shared__ double s_red[4][FISHER_ROWS];
  const int64_t row0 = (int64_t)blockIdx.x * FISHER_ROWS;
  const int tid = threadIdx.x;
  double racc[FISHER_ROWS];
#pragma unroll
  for (int r = 0; r < FISHER_ROWS; ++r) racc[r] = 0.0;
  for (int64_t c = tid; c < k; c += 256) {
    double cacc = 0.0;
#pragma unroll
    for (int r = 0; r < FISHER_ROWS; ++r) {
      const double s = row0 + r < d ? sqrt((double)F[(row0 + r) * k + c]) : 0.0;
      cacc += s;
      racc[r] += s;
    }
    colpart[(size_t)blockIdx.x * k + c] = cacc;
  }
#pragma unroll
  for (int r = 0; r < FISHER_ROWS; ++r) {
    double x = racc[r];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if ((tid & 63) == 0) s_red[tid >> 6][r] = x;
  }
  __syncthreads();
  if (tid < FISHER_ROWS && row0 + tid < d) rowsum[row0 + tid] = (s_red[0][tid] + s_red[1][tid]) + (s_red[2][tid] + s_red[3][tid]);
}

// Pass 2: every workgroup forms the grand total from the row sums in the same fixed order, then finishes its share
// of the outputs: row_w = a^2, col_w = (b / mean)^2 with a, b the row and column means of sqrt(F).
__global__ __launch_bounds__(256) void fisher_finalize_kernel(const double* __restrict__ rowsum,
                                                              const double* __restrict__ colpart, int64_t d, int64_t k,
                                                              int chunks, float* __restrict__ row_w,
                                                              float* __restrict__ col_w) {
  __shared__ double s_red[4];
  const int tid = threadIdx.x;
  double tot = 0.0;
  for (int64_t i = tid; i < d; i += 256) tot += rowsum[i];
  for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o);
  if ((tid & 63) == 0) s_red[tid >> 6] = tot;
  __syncthreads();
  const double mean = ((s_red[0] + s_red[1]) + (s_red[2] + s_red[3])) / ((double)d * (double)k);
  const int64_t gid = (int64_t)blockIdx.x * 256 + tid, stride = (int64_t)gridDim.x * 256;
  for (int64_t i = gid; i < d; i += stride) {
    const double a = rowsum[i] / (double)k;
    row_w[i] = (float)(a * a);
  }
  for (int64_t j = gid; j < k; j += stride) {
    double b = 0.0;
    for (int ch = 0; ch < chunks; ++ch) b += colpart[(size_t)ch * k + j];
    b = b / (double)d / mean;
    col_w[j] = (float)(b * b);
  }
}

size_t fisher_scratch_doubles(int64_t d, int64_t k) {
  return (size_t)d + (size_t)((d + FISHER_ROWS - 1) / FISHER_ROWS) * (size_t)k;
}

int launch_fisher_row_col(const float* F, int64_t d, int64_t k, double* scratch, float* row_w, float* col_w,
                          hipStream_t st) {
  const int64_t chunks = (d + FISHER_ROWS - 1) / FISHER_ROWS;
  if (chunks >= (1ll << 31)) return LQ_ERR_SHAPE;
  double* rowsum = scratch;
  double* colpart = scratch + d;
  hipLaunchKernelGGL(fisher_partial_kernel, dim3((unsigned)chunks), dim3(256), 0, st, F, d, k, rowsum, colpart);
  LQ_HIP_TRY(hipGetLastError());
  const int64_t want = (std::max(d, k) + 255) / 256;
  hipLaunchKernelGGL(fisher_finalize_kernel, dim3((unsigned)std::min<int64_t>(want, 256)), dim3(256), 0, st, rowsum,
                     colpart, d, k, (int)chunks, row_w, col_w);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

}  // namespace lq
