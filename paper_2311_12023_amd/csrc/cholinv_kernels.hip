// Cholesky factor of a Gram matrix and its inverse in one kernel (l = 16 NB = 32 .. 128), fp64: G = C C^T; out = C^-1 as a
// dense fp32 l x l matrix (zeros above the diagonal) that rotate_kernel then applies to the basis.
#include "dense_device.h"
#include "kernels.h"
#include "profiler.h"

namespace lq {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Blocks of 16 x 16, one workgroup of four wavefronts per problem.  With U = C^T and the inverse X = C^-1, step J factors
// the diagonal block (G_JJ = C_JJ C_JJ^T, D = C_JJ^-1), scales the row, U_Jb = D G_Jb (b > J) and X_Ja = D S_Ja (a < J,
// X_JJ = D), and updates what lies beyond it: G_ab -= U_Ja^T U_Jb (J < a <= b) and S_ba -= U_Jb^T X_Ja (a <= J < b).  G_ab
// and S_ba are needed one after the other, so the pair (a, b) has one slot, an MFMA accumulator of the wavefront that
// owns it (pair p belongs to wavefront p mod 4).  All products contract over the rows of block J, and the accumulator layout
// of v_mfma_f64_16x16x4_f64 (register r of a lane: row 4 r + lane / 16, column lane % 16) is then the layout of
// either operand: blocks go from accumulators through LDS into operands as they are.
// The diagonal block is factored by every wavefront for itself, lane i of each 16 holding row i: L D L^T without square
// roots in the chain (a pivot's reciprocal, the multipliers, the next pivot), in place as in Gauss-Jordan elimination:
// column j of the matrix gives way to column j of the inverse of L.  The serial chain is 16 short steps per block and two
// barriers, against a barrier, a reciprocal square root and two LDS round trips per column before (one problem, l = 128 54
// -> 34 us, l = 96 35 -> 21, l = 64 20 -> 12, l = 32 9.5 -> 5.7).
// A pivot is compared with the row's own squared norm, not with the largest one (see cholesky_kernel); one that is not
// positive (dependent direction) zeroes that row of C^-1, which removes the direction.

template <int J>
__device__ __forceinline__ double row_broadcast(double x) { return dpp_move<0x150 + J>(x); }     // row_newbcast: lane J of each 16

// x_m += f * (x_m of lane J of each 16), m < 5: the broadcast is part of the fp64 instruction, which the compiler, having only
// the 32-bit move as a builtin, spells as two moves each.  The wait states are those between the instruction that wrote a
// register and one that reads it across lanes.
template <int J>
__device__ __forceinline__ void add_multiple(double& x0, double& x1, double& x2, double& x3, double& x4, double f) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %1, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %2, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %3, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, %4, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf"
      : "+&v"(x0), "+&v"(x1), "+&v"(x2), "+&v"(x3), "+&v"(x4)
      : "v"(f), "i"(J));
}

// a: row i = lane % 16 of a symmetric 16 x 16 block; thr: what its pivot has to exceed.  On return row i of the inverse of
// the Cholesky factor (entries past the diagonal zero).
__device__ __forceinline__ void invert_block(double (&a)[16], double thr, int i) {
  double pivot = 0.0;
  for_each_block<16>([&](auto step) {
    constexpr int j = decltype(step)::value;
    if (i == j) pivot = a[j];
    const double x = a[j], r = row_broadcast<j>(x > thr ? rcp64(x) : 0.0);
    const double f = i > j ? -x * r : 0.0;
    for_each_block<3>([&](auto part) {                         // the next pivot's column first
      constexpr int k = j + 1 + 5 * decltype(part)::value;
      add_multiple<j>(a[k % 16], a[(k + 1) % 16], a[(k + 2) % 16], a[(k + 3) % 16], a[(k + 4) % 16], f);
    });
    a[j] = i == j ? 1.0 : f;
  });
  const double scale = pivot > thr ? rsqrt64(pivot) : 0.0;
  for_each_block<16>([&](auto column) {
    constexpr int k = decltype(column)::value;
    a[k] = k <= i ? a[k] * scale : 0.0;
  });
}

template <int NB>
__global__ __launch_bounds__(256, 2) void cholinv_kernel(const double* __restrict__ Gall, float* __restrict__ Cinvall) {
  constexpr int l = 16 * NB, PAIRS = NB * (NB + 1) / 2, SLOTS = (PAIRS + 3) / 4, PD = 18;
  __shared__ double s_left[NB][4][64];         // -U_Jb, b > J: left operands
  __shared__ double s_right[NB][4][64];        // U_Jb, b > J; X_Ja, a <= J: right operands
  __shared__ __attribute__((aligned(16))) double s_block[16 * PD];
  __shared__ double s_thr[l];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const double* G = Gall + (size_t)blockIdx.x * l * l;
  __builtin_amdgcn_s_setprio(3);               // a serial chain that shares the compute unit with streaming kernels
  doublex4 acc[SLOTS];
  int ra[SLOTS], rb[SLOTS];                    // the pair of each slot, a <= b (past the end: none is ever active)
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int p = w + 4 * s;
    int b = 0, a = p;
    while (a > b) { a -= b + 1; ++b; }
    const bool there = p < PAIRS;
    ra[s] = there ? a : -1; rb[s] = there ? b : -1;
    acc[s] = doublex4{0, 0, 0, 0};
    if (there) {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[s][r] = G[(size_t)(16 * a + 4 * r + q) * l + 16 * b + n];
    }
  }
  if (threadIdx.x < l) s_thr[threadIdx.x] = 1e-12 * G[(size_t)threadIdx.x * l + threadIdx.x];
  if (w == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) s_block[(4 * r + q) * PD + n] = acc[0][r];
  }
#pragma nounroll
  for (int J = 0; J < NB; ++J) {
    __syncthreads();
    double row[16];
#pragma unroll
    for (int k = 0; k < 16; k += 2) {
      const double2 v = *reinterpret_cast<const double2*>(s_block + n * PD + k);
      row[k] = v.x; row[k + 1] = v.y;
    }
    int i = n;
    asm volatile("" : "+v"(i));                // the comparisons with it stay in the loop instead of filling the scalar registers
    invert_block(row, s_thr[16 * J + n], i);
    double d[4];                               // left operand: row n, columns 4 t + q
#pragma unroll
    for (int t = 0; t < 4; ++t)
      d[t] = q & 2 ? (q & 1 ? row[4 * t + 3] : row[4 * t + 2]) : (q & 1 ? row[4 * t + 1] : row[4 * t]);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      if (ra[s] == J || rb[s] == J) {          // row J of U or of X
        const bool diagonal = ra[s] == rb[s], upper = rb[s] > J;
        doublex4 x = {0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < 4; ++t)
          x = __builtin_amdgcn_mfma_f64_16x16x4f64(d[t], diagonal ? (4 * t + q == n ? 1.0 : 0.0) : acc[s][t], x, 0, 0, 0);
        const int other = upper ? rb[s] : ra[s];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s_right[other][r][lane] = x[r];
          if (upper) s_left[other][r][lane] = -x[r];
          acc[s][r] = upper ? 0.0 : x[r];
        }
      }
    }
    if (J + 1 == NB) break;
    __syncthreads();
    double x[2][4], y[2][4];
    auto fetch = [&](int s, double (&xs)[4], double (&ys)[4]) {      // slots past the end and finished ones read block 0 or J
      const int a = ra[s], b = rb[s], left = a > J ? a : b, right = a > J ? b : a;
#pragma unroll
      for (int t = 0; t < 4; ++t) { xs[t] = s_left[left < 0 ? 0 : left][t][lane]; ys[t] = s_right[right < 0 ? 0 : right][t][lane]; }
    };
    fetch(0, x[0], y[0]);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      if (s + 1 < SLOTS) fetch(s + 1, x[(s + 1) & 1], y[(s + 1) & 1]);
      if (rb[s] > J) {
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s & 1][t], y[s & 1][t], acc[s], 0, 0, 0);
        if (ra[s] == J + 1 && rb[s] == J + 1) {            // the next diagonal block
#pragma unroll
          for (int r = 0; r < 4; ++r) s_block[(4 * r + q) * PD + n] = acc[s][r];
        }
      }
    }
  }
  float* out = Cinvall + (size_t)blockIdx.x * l * l;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    if (rb[s] < 0) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * r + q;
      out[(size_t)(16 * rb[s] + row) * l + 16 * ra[s] + n] = (float)acc[s][r];
      if (ra[s] != rb[s]) out[(size_t)(16 * ra[s] + row) * l + 16 * rb[s] + n] = 0.0f;
    }
  }
}

bool cholinv_supported(int l) { return l % 32 == 0 && l >= 32 && l <= 128; }

int launch_cholinv(const double* G, int l, float* Cinv, int batch, hipStream_t st) {
  prof::Scope ps(prof::CHOLESKY, st, (double)l * l * 12.0 * batch);
  switch (l / 32) {
    case 1: hipLaunchKernelGGL(cholinv_kernel<2>, dim3(batch), dim3(256), 0, st, G, Cinv); break;
    case 2: hipLaunchKernelGGL(cholinv_kernel<4>, dim3(batch), dim3(256), 0, st, G, Cinv); break;
    case 3: hipLaunchKernelGGL(cholinv_kernel<6>, dim3(batch), dim3(256), 0, st, G, Cinv); break;
    case 4: hipLaunchKernelGGL(cholinv_kernel<8>, dim3(batch), dim3(256), 0, st, G, Cinv); break;
    default: return LQ_ERR_ARG;
  }
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

}  // namespace lq
