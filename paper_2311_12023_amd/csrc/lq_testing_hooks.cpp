// Test hooks (include/lq_testing.h): single kernels of the randomized SVD, the host evaluation of the code search and
// the capture of one configuration's iterate inside the sweep.  This file is compiled only into the testing build of
// the library (liblq_hip_testing.so, everything compiled with -DLQ_TESTING_HOOKS); the product library exports none of it.
#include <cmath>

#include "../../include/lq_testing.h"
#include "dense_device.h"
#include "kernels.h"
#include "nf_device.h"
#include "testing_capture.h"

namespace lq {
size_t lds_limit_for_tests();
namespace testing {
Capture& capture() {
  static thread_local Capture c;
  return c;
}
}  // namespace testing
}  // namespace lq

using namespace lq;

static __device__ double g_eig_work[lq::sym_eig_work_doubles(128)];

extern "C" {

int lq_test_capture_iterate(int cfg_index, int iter, float* Q_dense, double* sigma_next) {
  testing::Capture& c = testing::capture();
  c = testing::Capture();
  if (cfg_index < 0) return LQ_OK;                      // disarm
  if (iter < 1 || !Q_dense) return LQ_ERR_ARG;
  c.armed = true; c.cfg = cfg_index; c.iter = iter; c.Q = Q_dense; c.sigma = sigma_next;
  return LQ_OK;
}

int lq_test_wide_gemm(int mode, int l, int64_t big, int64_t K, const float* X, int64_t ldx, const float* A,
                      int64_t lda, float* C, int64_t ldc, int batch, int workgroups, float* part, size_t part_floats,
                      int precision, void* stream) {
  if (!X || !A || !C) return LQ_ERR_NULL;
  if ((precision != 0 && precision != 1) || workgroups < -32768 || workgroups > 32768 || batch < 1) return LQ_ERR_ARG;
  const size_t sA = (size_t)(mode == MODE_NT ? big : K) * lda;
  return launch_wide_gemm(mode, l, big, K, X, ldx, (size_t)l * ldx, A, lda, sA, C, ldc, (size_t)l * ldc, batch, part,
                          part_floats, (hipStream_t)stream, precision, workgroups);
}

int lq_test_wide_gemm_f16(int mode, int l, int64_t big, int64_t K, const float* X, int64_t ldx, const uint16_t* A,
                          const uint8_t* A_lo, int64_t lda, float* C, int64_t ldc, int batch, int workgroups, float* part, size_t part_floats,
                          float x_scale, const double* lam0, float out_scale, void* stream) {
  if (!X || !A || !C) return LQ_ERR_NULL;
  if (workgroups < -32768 || workgroups > 32768 || batch < 1) return LQ_ERR_ARG;
  const size_t sA = (size_t)(mode == MODE_NT ? big : K) * lda;
  return launch_wide_gemm_f16(mode, l, big, K, X, ldx, (size_t)l * ldx, A, A_lo, lda, sA, C, ldc, (size_t)l * ldc, batch, part,
                              part_floats, x_scale, lam0, 1, out_scale, (hipStream_t)stream, workgroups);
}

size_t lq_test_wide_gemm_part_floats(int l, int workgroups) {
  if (l % 32 != 0 || l < 32 || l > 256) return 0;
  return gemm_part_floats(l, workgroups);
}

int lq_test_orthonormalize(float* X, int l, int64_t m, int64_t ldx, double* scratch, float* alt, void* stream) {
  if (!X || !scratch) return LQ_ERR_NULL;
  if (l % 32 || l < 32 || l > 256) return LQ_ERR_ARG;
  double* G = scratch;
  double* part = scratch + (size_t)l * l;
  LQ_TRY(launch_gram(X, l, m, ldx, 0, part, (size_t)16 * l * l, G, 1, (hipStream_t)stream));
  if (cholinv_supported(l) && alt) {
    float* Cinv = reinterpret_cast<float*>(part);       // the Gram partials are dead by now
    LQ_TRY(launch_cholinv(G, l, Cinv, 1, (hipStream_t)stream));
    LQ_TRY(launch_rotate(l, Cinv, 0, true, X, alt, ldx, 0, nullptr, nullptr, 0, 0, 1, (hipStream_t)stream));
    LQ_HIP_TRY(hipMemcpyAsync(X, alt, (size_t)l * ldx * sizeof(float), hipMemcpyDeviceToDevice, (hipStream_t)stream));
    return LQ_OK;
  }
  LQ_TRY(launch_cholesky(G, l, 1, (hipStream_t)stream));
  return launch_trsm(G, l, X, m, ldx, 0, 1, (hipStream_t)stream);
}

int lq_test_sym_eig(double* G, int l, float* Ut, double* lambda, double* scratch, void* stream) {
  if (!G || !Ut || !lambda || !scratch) return LQ_ERR_NULL;
  if (l % 2 || l < 2 || l > 256) return LQ_ERR_ARG;
  return launch_jacobi_eig(G, l, scratch, Ut, lambda, 1, (hipStream_t)stream);
}

int lq_test_sym_eig_fast(const double* G, int l, float* Ut, double* lambda, void* stream) {
  if (!G || !Ut || !lambda) return LQ_ERR_NULL;
  if (!sym_eig_supported(l)) return LQ_ERR_ARG;
  void* work = nullptr;
  LQ_HIP_TRY(hipGetSymbolAddress(&work, HIP_SYMBOL(g_eig_work)));
  return launch_sym_eig(G, l, static_cast<double*>(work), Ut, lambda, 1, (hipStream_t)stream);
}

int lq_test_sym_eig_batch(const double* G, int l, int batch, double* work, float* Ut, double* lambda, void* stream) {
  if (!G || !work || !Ut || !lambda) return LQ_ERR_NULL;
  if (!sym_eig_supported(l) || batch < 1) return LQ_ERR_ARG;
  return launch_sym_eig(G, l, work, Ut, lambda, batch, (hipStream_t)stream);
}

int lq_test_gram(const float* X, int l, int64_t m, int64_t ldx, size_t stride, double* part, size_t part_doubles, double* G,
                 int batch, void* stream) {
  if (!X || !part || !G) return LQ_ERR_NULL;
  return launch_gram(X, l, m, ldx, stride, part, part_doubles, G, batch, (hipStream_t)stream);
}

int lq_test_rotate(int l, const float* U, size_t strideU, int lower, const float* A0, float* C0, int64_t ld0, size_t stride0,
                   const float* A1, float* C1, int64_t ld1, size_t stride1, int batch, void* stream) {
  if (!U || !A0 || !C0 || (A1 && !C1)) return LQ_ERR_NULL;
  return launch_rotate(l, U, strideU, lower != 0, A0, C0, ld0, stride0, A1, C1, ld1, stride1, batch, (hipStream_t)stream);
}

int lq_test_filter_step(float* X, float a, const float* Y, float b, const float* Z, float c, const float* L, int l, int locked,
                        int64_t m, int64_t ldx, void* stream) {
  if (!X || !L) return LQ_ERR_NULL;
  if (l < 1 || locked > l || m < 1 || ldx < m) return LQ_ERR_ARG;
  return launch_filter_step(X, a, Y, b, Z, c, L, l, locked, m, ldx, (hipStream_t)stream);
}

int lq_test_filter_step_packed(float* X, float a, const float* Y, float b, const float* Z, float c, const float* L, int l,
                               int locked, int64_t m, int64_t ldx, const float* part, int ranges, uint16_t* packed,
                               void* stream) {
  if (!X || !L) return LQ_ERR_NULL;
  if (l < 1 || locked > l || m < 1 || ldx < m) return LQ_ERR_ARG;
  return launch_filter_step(X, a, Y, b, Z, c, L, l, locked, m, ldx, (hipStream_t)stream, part, ranges, packed);
}

int lq_test_pack(int l, const float* X, int64_t ldx, uint16_t* packed, void* stream) {
  if (!X || !packed) return LQ_ERR_NULL;
  return launch_column_sum(l, X, ldx, 1, ldx, nullptr, 0, packed, (hipStream_t)stream);
}

int lq_test_column_gemm(int mode, int l, int64_t big, int64_t K, const float* X, int64_t ldx, const float* A, int64_t lda,
                        float* C, int64_t ldc, uint16_t* C_packed, int nt, int ranges, float* scratch, void* stream) {
  if (!X || !A || !C || !scratch) return LQ_ERR_NULL;
  if (big < 1 || ldc < (big + 63) / 64 * 64 || ldx < K || !column_gemm_supported(l)) return LQ_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const ColumnSplit split = nt ? ColumnSplit{nt, ranges} : column_gemm_split(l, big, K);
  uint16_t* xp = reinterpret_cast<uint16_t*>(scratch);
  float* part = scratch + (size_t)l * ldx;
  LQ_TRY(launch_column_sum(l, X, ldx, 1, ldx, nullptr, 0, xp, st));
  LQ_TRY(launch_column_gemm(mode, l, big, K, xp, A, lda, split, C, ldc, C_packed, part, st));
  if (split.ranges == 1) return LQ_OK;
  return launch_column_sum(l, part, (big + 63) / 64 * 64, split.ranges, big, C, ldc, C_packed, st);
}

int lq_test_lincomb3(float* X, float a, const float* Y, float b, const float* Z, float c, int l, int64_t ldx, void* stream) {
  if (!X || !Y) return LQ_ERR_NULL;
  if (l < 1 || ldx < 4 || ldx % 4) return LQ_ERR_ARG;
  return launch_filter_step(X, a, Y, b, Z, c, nullptr, l, 0, ldx, ldx, (hipStream_t)stream);
}

int lq_test_deflate_rows(float* X, const float* L, int l, int locked, int64_t m, int64_t ldx, void* stream) {
  if (!X || !L) return LQ_ERR_NULL;
  if (l < 1 || m < 1 || m > ldx || locked > l) return LQ_ERR_ARG;
  return launch_deflate_rows(X, L, l, locked, m, ldx, (hipStream_t)stream);
}

int lq_test_ritz_residual(const float* G, const float* Y, const double* lam, int rows, int64_t m, int64_t ldx, double* res,
                          void* stream) {
  if (!G || !Y || !lam || !res) return LQ_ERR_NULL;
  if (rows < 1 || m < 1 || m > ldx) return LQ_ERR_ARG;
  return launch_ritz_residual(G, Y, lam, rows, m, ldx, res, (hipStream_t)stream);
}

int lq_test_bucket_code(int bits, float x) {
  const int slot = bits_slot(bits);
  if (slot < 0) return -1;
  const HostTables& t = host_tables();
  // the search of the stand-alone quantizer for 4 and 8 bits: bucket table, then one comparison (two for 8 bits); for 2 and 3
  // bits it counts thresholds, which is the definition
  int j = (int)std::fmaf(x, 256.0f, 256.0f);
  if (!(std::fmaf(x, 256.0f, 256.0f) >= 0.0f)) j = 0;   // NaN and negatives as the device's conversion treats them
  j = j < 0 ? 0 : (j > 513 ? 513 : j);
  const int c0 = t.lut[slot][j < 511 ? j : 511];
  if (bits <= 4) return c0 + (x >= t.thr[slot][c0]);          // one threshold per bucket at most
  return c0 + (x >= t.thr[slot][c0]) + (x >= t.thr[slot][c0 + 1]);
}

int lq_test_search_code(int bits, float x) {
  const int slot = bits_slot(bits);
  if (slot < 0) return -1;
  const HostTables& t = host_tables();
  // entries past the end of the width's table: found as if they held this code
  constexpr uint32_t outside = 1u << 16;
  SearchEntry table[4 * search_buckets(8)];
  for (int j = 0; j < 4 * search_buckets(8); ++j)
    table[j] = j < search_entries(bits) ? t.search[slot][j] : SearchEntry{HUGE_VALF, outside};
  const uint32_t c = bits == 8 ? search_code<8>(table, x) : search_code<4>(table, x);
  return c >= outside ? -2 : (int)c;
}

float lq_test_sigma_by_reciprocal(float v, int levels) {
  return sigma_by_reciprocal(v, (float)levels, 1.0f / (float)levels);
}

int lq_test_search_points(double flo, int elo, double fhi, int ehi, int wanted, double q, double* points) {
  const SearchPoints at = search_points(flo, elo, fhi, ehi, wanted != 0, q);
  points[0] = at.a; points[1] = at.b;
  return at.secant;
}

int lq_test_rows_finish(int64_t m, int64_t N, int rank) { return rows_finish_preferred(m, N, rank); }

size_t lq_test_lds_limit(void) { return lds_limit_for_tests(); }

}  // extern "C"
